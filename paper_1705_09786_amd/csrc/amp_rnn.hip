// Persistent kernel of the variable-length RNN.
#include <hip/hip_runtime.h>
#include "amp_worker.hip.h"
#include "amp_batch.hip.h"
#include "amp_tree.hip.h"
#include "amp_rnn.hip.h"
#include "amp_rnn_cell.hip.h"

static __device__ __forceinline__ void rnn_worker(const GQ AmpDev* D, const GQ WorkerDev* W) {
  if (W->role == ROLE_RNN_CELL) {
    // weights in registers wherever the rest fits the LDS (the threshold and the table decide; the choice is made anew
    // in every launch, and what is carried over between launches has one layout)
    if (rnn_reg_fits(D, W)) {
      const int opt = D->node[W->node].opt;
      if (D->node_replicas > 1 && D->sync_every > 0)
        opt == 0 ? role_rnn_cell_reg<0, true>(D, W) : opt == 1 ? role_rnn_cell_reg<1, true>(D, W) : role_rnn_cell_reg<2, true>(D, W);
      else
        opt == 0 ? role_rnn_cell_reg<0, false>(D, W) : opt == 1 ? role_rnn_cell_reg<1, false>(D, W) : role_rnn_cell_reg<2, false>(D, W);
    }
    // hidden = emb = 128 (8 row blocks, 16 column groups) has products with fixed trip counts
    else if (D->node[1].rows == 128 && D->node[1].cols == 256 && D->node[1].seg0 == 128)
      role_rnn_cell<8, 16>(D, W);
    else
      role_rnn_cell<0, 0>(D, W);
  } else if (rnn_out_fits(D)) {
    role_rnn_out_batch(D, W);
  } else {
    role_rnn_out(D, W);
  }
}

AMP_PERSISTENT_KERNEL(rnn, false, rnn_worker(D, W);)
