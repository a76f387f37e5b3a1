// Persistent kernel of the binary Tree-LSTM.
#include <hip/hip_runtime.h>
#include "amp_worker.hip.h"
#include "amp_batch.hip.h"
#include "amp_tree.hip.h"

static __device__ __forceinline__ void tree_worker(const GQ AmpDev* D, const GQ WorkerDev* W) {
  switch (W->role) {
    case ROLE_TREE_LOOKUP: role_tree_lookup(D, W); break;
    case ROLE_TREE_LEAF:
    case ROLE_TREE_BRANCH: {
      // hidden 150 / embedding 300 (nineteen 16-column groups) split into tiles of six, four or three 16-row blocks
      // (5 + 8 tiles, the fewest that fit LDS; 8 leaf tiles; 16 branch tiles) has instantiations with fixed trip counts
      const GQ NodeDev& nd = D->node[W->node];
      const int rp = amp_round16(nd.nblocks * W->nu), cl = (nd.cols / nd.seg) * nd.segp;
      const bool c19 = amp_round16(cl) == 304;
      if (W->role == ROLE_TREE_LEAF) {
        if (W->aux == 1) role_tree_cell<false, 0, 0, true>(D, W);
        else if (c19 && rp == 96) role_tree_cell<false, 6, 19, false>(D, W);
        else if (c19 && rp == 64) role_tree_cell<false, 4, 19, false>(D, W);
        else if (c19 && rp == 48) role_tree_cell<false, 3, 19, false>(D, W);
        else role_tree_cell<false, 0, 0, false>(D, W);
      } else {
        if (W->aux == 1) role_tree_cell<true, 0, 0, true>(D, W);
        else if (c19 && rp == 96) role_tree_cell<true, 6, 19, false>(D, W);
        else if (c19 && rp == 64) role_tree_cell<true, 4, 19, false>(D, W);
        else if (c19 && rp == 48) role_tree_cell<true, 3, 19, false>(D, W);
        else role_tree_cell<true, 0, 0, false>(D, W);
      }
      break;
    }
    case ROLE_TREE_OUT: role_tree_out(D, W); break;
    default: break;
  }
}

AMP_PERSISTENT_KERNEL(tree, tree_worker(D, W);)
