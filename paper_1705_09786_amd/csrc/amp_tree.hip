// Persistent kernel of the binary Tree-LSTM.
#include <hip/hip_runtime.h>
#include "amp_worker.hip.h"
#include "amp_batch.hip.h"
#include "amp_tree.hip.h"
#include "amp_tree_cell.hip.h"
#include "amp_tree_out.hip.h"

template <bool BR, int GU>
static __device__ __forceinline__ void tree_cell_opt(const GQ AmpDev* D, const GQ WorkerDev* W) {
  const int opt = D->node[W->node].opt;
  if (opt == 0) role_tree_cell_lds<BR, GU, 0>(D, W);
  else if (opt == 1) role_tree_cell_lds<BR, GU, 1>(D, W);
  else role_tree_cell_lds<BR, GU, 2>(D, W);
}

template <bool BR>
static __device__ __forceinline__ void tree_cell_worker(const GQ AmpDev* D, const GQ WorkerDev* W) {
  const GQ NodeDev& nd = D->node[W->node];
  const int cl = ((nd.cols - nd.seg0) / nd.seg + 1) * nd.segp, rows = amp_round16(nd.nblocks * W->nu);
  if (W->aux == 1) return role_tree_cell<BR, 0, 0, true>(D, W);
  if (W->aux == 0) {
    // hidden 150 / embedding 300 on 5 + 8 tiles, the fewest that fit the LDS: products with fixed trip counts
    if (rows == 96 && amp_round16(cl) == 304) return role_tree_cell<BR, 6, 19, false>(D, W);
    return role_tree_cell<BR, 0, 0, false>(D, W);
  }
  // units of 16 rows x 64 columns a wave owns of the gradient
  const int units = (rows >> 4) * ((amp_round16(cl) + 63) >> 6);
  if (units <= 8) tree_cell_opt<BR, 1>(D, W);
  else if (units <= 16) tree_cell_opt<BR, 2>(D, W);
  else if (units <= 24) tree_cell_opt<BR, 3>(D, W);
  else tree_cell_opt<BR, 4>(D, W);
}

static __device__ __forceinline__ void tree_worker(const GQ AmpDev* D, const GQ WorkerDev* W) {
  switch (W->role) {
    case ROLE_TREE_LOOKUP: role_tree_lookup(D, W); break;
    case ROLE_TREE_LEAF: tree_cell_worker<false>(D, W); break;
    case ROLE_TREE_BRANCH: tree_cell_worker<true>(D, W); break;
    case ROLE_TREE_OUT: {
      // groups of four columns of the gradient, dealt to 384 threads; the host admits up to 6144 elements in 64 rows
      const int n = D->n_class * ((D->hidden + 3) >> 2);
      if (n <= 384) role_tree_out<1>(D, W);
      else if (n <= 2 * 384) role_tree_out<2>(D, W);
      else role_tree_out<5>(D, W);
      break;
    }
    default: break;
  }
}

AMP_PERSISTENT_KERNEL(tree, false, tree_worker(D, W);)
