// Tree-LSTM workers (Section 6, Tree-LSTM paragraph): lookup, leaf cell,
// branch cell, output layer with a softmax loss at every tree node.
//
// Leaf and branch cells are split over several workgroups ("tiles", Section
// 5.1); the tiles of a cell read the same ring in the same order and cut
// their batches at the same updates, so they act as one node with one event
// order.  Tile t owns hidden units [u0, u0+nu) of every gate, computes those
// units' h and c entirely, and contributes a partial W^T delta over all
// input columns on the way back.
//
// A worker takes up to 64 waiting messages at once.  Cells whose weights leave the LDS room for a batch's inputs are
// role_tree_cell_lds (amp_tree_cell.hip.h), which keeps the node's gradient in registers.  In role_tree_cell the inputs of
// the forward product go from the slot storage in HBM straight into the matrix cores' operand registers (rows there are
// padded to multiples of 4 floats so that every 16-byte fetch is aligned); each backward message appends its (delta,
// input) pair to the tile's pending list in HBM, and the update forms the accumulated gradient from that list on the
// matrix cores.  In both the input gradient goes from the accumulators straight back to HBM.
//
// Slot storage (s = slot, n = tree node, l = leaf; Hp, Ep = H, E rounded up to 4;
// padding entries stay zero):
//   buf[0] xin  [s][l][Ep]       embedding recorded by the lookup's forward
//   buf[1] hc   [s][n][2][Hp]    node output: h then c
//   buf[2] gate [s][n][6][H]     gate activations and tanh(c) recorded at forward
//   buf[3] gout [s][n][H]        dh from the output layer
//   buf[4] gpar [s][n][TB][Hp]   dh partials from the parent's tiles
//   buf[5] gc   [s][n][H]        dc from the parent
//   buf[6] gx   [s][l][TL][Ep]   dx partials from the leaf tiles
//   buf[7] cnt  [s][n][4] (int)  arrival counters: tiles done / children done /
//                                gradient parts / leaf-tile dx parts
//   buf[10] lookup: tokens of the gradients waiting for the next update
//   buf[11] lookup: their gradient rows [AMP_TREE_LOOKUP_MAX_MUF][E]
#pragma once

struct TreeBufs {
  GQ float *xin, *hc, *gate, *gout, *gpar, *gc, *gx;
  GQ int* cnt;
  int H, Hp, E, Ep, NNmax, Lmax, TL, TB;
  __device__ __forceinline__ long long node(int s, int n) const { return (long long)s * NNmax + n; }
  __device__ __forceinline__ long long leaf(int s, int l) const { return (long long)s * Lmax + l; }
  __device__ __forceinline__ unsigned node32(int s, int n) const { return (unsigned)(s * NNmax + n); }   // nodes of all slots < 2^31
};

__device__ __forceinline__ TreeBufs tree_bufs(const GQ AmpDev* D) {
  TreeBufs b;
  b.xin = uni_gq<float>(D->buf[0]);
  b.hc = uni_gq<float>(D->buf[1]);
  b.gate = uni_gq<float>(D->buf[2]);
  b.gout = uni_gq<float>(D->buf[3]);
  b.gpar = uni_gq<float>(D->buf[4]);
  b.gc = uni_gq<float>(D->buf[5]);
  b.gx = uni_gq<float>(D->buf[6]);
  b.cnt = uni_gq<int>(D->buf[7]);
  b.H = uni(D->hidden);
  b.Hp = amp_round4(b.H);
  b.E = uni(D->emb);
  b.Ep = amp_round4(b.E);
  b.Lmax = uni(D->max_len);
  b.NNmax = 2 * b.Lmax - 1;
  b.TL = uni(D->tiles_leaf);
  b.TB = uni(D->tiles_branch);
  return b;
}

// Ring numbers of the tree model.
#define TR_LOOKUP 1
#define TR_LEAF 2
#define TR_BRANCH 3
#define TR_OUT 4

__device__ __forceinline__ bool code_is_b(unsigned c) { return (c & MSG_DIR_B) != 0; }

// What a worker keeps of its descriptor and of the rings it posts to, read once (into scalar registers).
struct WorkerRegs {
  int node, tile, ntiles, kb, train;
  unsigned log_cap;
  GQ unsigned long long* log;
  Ring ctl, lookup, leaf, branch, out;   // the tree model's rings
};

__device__ __forceinline__ WorkerRegs worker_regs(const GQ AmpDev* D, const GQ WorkerDev* W) {
  WorkerRegs w;
  w.node = uni(W->node);
  w.tile = uni(W->tile);
  w.ntiles = uni(W->ntiles);
  w.kb = uni(W->kb);
  w.train = uni(D->train);
  w.log_cap = uni(W->log_cap);
  w.log = uni_gq<unsigned long long>(W->log);
  w.ctl = ring_regs(D, 0);
  w.lookup = ring_regs(D, 1);
  w.leaf = ring_regs(D, 2);
  w.branch = ring_regs(D, 3);
  w.out = ring_regs(D, 4);
  return w;
}


// What the controller wrote for slot s at admission: admission number, leaves, node offset, token offset.
__device__ __forceinline__ v4i tree_slot(const GQ int* smeta, int s) { return *(const GQ v4i*)(smeta + 4 * s); }
// left, right, parent * 2 + side (-1 for the root), label of node n of the instance whose nodes start at noff
__device__ __forceinline__ v4i tree_node(const GQ int* tnode, int noff, int n) {
  return *(const GQ v4i*)(tnode + 4 * (long long)(noff + n));
}

// One wave, all 64 lanes (k = lane), after lanes k < n have written M.aux[k]: positions
// of the batch's forward and backward messages, and the event record (tile 0 only).
__device__ __forceinline__ void batch_split_and_log(const GQ AmpDev* D, const WorkerRegs& W, BatchMsg& M, int n, int node) {
  const int k = threadIdx.x & 63;
  const bool in = k < n, isb = in && M.aux[k] != 0;
  const unsigned long long mb = __ballot(isb), mf = __ballot(in && !isb);
  const unsigned long long lt = (1ull << k) - 1ull;
  if (isb) M.bidx[__popcll(mb & lt)] = k;
  if (in && !isb) M.fidx[__popcll(mf & lt)] = k;
  if (k == 0) {
    M.nF = __popcll(mf);
    M.nB = __popcll(mb);
  }
  if (W.log_cap && W.tile == 0) {
    const unsigned base = s_logn;
    if (base + (unsigned)n > W.log_cap) {
      if (k == 0) raise_abort(D, ABORT_LOG_FULL, blockIdx.x);
    } else {
      if (in) {
        const unsigned long long tail = ((unsigned long long)M.seq[k] << 32) | ((unsigned)node << 20) | ((unsigned)M.n[k] & 0xfffffu);
        W.log[base + k] = tail | ((unsigned long long)(isb ? 1 : 0) << 28);
      }
      if (k == 0) s_logn = base + (unsigned)n;
    }
  }
}

// What a lane needs of its message to publish it.
struct TreePost {
  int s, n, a, b, par, L;
  bool in, fwd;
};
__device__ __forceinline__ TreePost tree_post_of(const BatchMsg& M, int r, bool in, bool fwd) {
  TreePost p;
  p.s = M.s[r];
  p.n = M.n[r];
  p.a = M.a[r];
  p.b = M.b[r];
  p.par = M.par[r];
  p.L = M.L[r];
  p.in = in;
  p.fwd = fwd;
  return p;
}

// A cell tile's batch is written: joins and posts, one message per lane of the calling wave (all 64 lanes), after a release
// fence.  Forward: when all tiles have done node n, its [h; c] goes to the output layer and, through Isu / Concat, to its
// parent, which fires once both children are there.  Backward: a part for each child (branch cells) or for the
// embedding's gradient (leaf cells) has arrived.  Every step of this is an atomic's round trip, so the lanes take each step
// together: the arrivals of all messages, then the parents' arrivals beside one reservation per ring (a lane for each
// ring), then the entries.  (Message by message, join after join, a batch whose tile arrives last took 3.4 us here; its
// node waits for that tile.  Without in_flight, and with the rings' tails picked from the struct in memory, the compiler
// waited for each fetch by itself and read the tail from scratch: 2,136 trees 41.8 ms instead of 39.2, one tree at a time forward
// 10.8 ms per 100 instead of 10.3; 16 replicas, whose fetches stay inside a die, 10.16 instead of 10.26.)
template <bool BR>
__device__ __forceinline__ void tree_publish(const WorkerRegs& W, const TreeBufs& B, const TreePost& p) {
  const int lane = threadIdx.x & 63;
  const unsigned long long lt = (1ull << lane) - 1ull;
  const bool f = p.in && p.fwd, b = p.in && !p.fwd;
  GQ int* c0 = B.cnt + B.node(p.s, BR && b ? p.a : p.n) * 4 + (p.fwd ? 0 : BR ? 2 : 3);
  GQ int* c1 = B.cnt + B.node(p.s, BR && b ? p.b : p.n) * 4 + 2;
  const Ring& down = BR ? W.leaf : W.lookup;
  GQ unsigned *const tail_out = W.out.tail, *const tail_down = down.tail, *const tail_branch = W.branch.tail;
  int o0 = 0, o1 = 0, o2 = 0;
  if (p.in) o0 = join_add(c0);
  if (BR && b) o1 = join_add(c1);
  in_flight(o0, o1);
  const bool d0 = p.in && o0 + 1 == (p.fwd ? W.ntiles : BR ? 1 + B.TB : B.TL);
  const bool d1 = BR && b && o1 + 1 == 1 + B.TB;
  // the parent's other child
  const bool up = f && d0 && p.par >= 0;
  GQ int* cp = B.cnt + B.node(p.s, up ? p.par >> 1 : p.n) * 4 + 1;
  const bool leaf0 = b && d0 && (!BR || p.a < p.L), leaf1 = d1 && p.b < p.L;   // leaf cells: to the lookup
  const bool br0 = b && d0 && !leaf0, br1 = d1 && !leaf1;
  const unsigned long long mo = __ballot(f && d0), ml0 = __ballot(leaf0), ml1 = __ballot(leaf1), mb0 = __ballot(br0), mb1 = __ballot(br1);
  const unsigned want = lane == 0 ? __popcll(mo) : lane == 1 ? __popcll(ml0) + __popcll(ml1) : lane == 2 ? __popcll(mb0) + __popcll(mb1) : 0u;
  GQ unsigned* tail = lane == 0 ? tail_out : lane == 1 ? tail_down : tail_branch;
  unsigned t = 0;
  if (up) o2 = join_add(cp);
  if (want) t = __hip_atomic_fetch_add(tail, want, __ATOMIC_RELAXED, AGENT);
  in_flight(o2, t);
  // (the counters are cleared only here: a fetch would wait for the stores in front of it)
  const bool d2 = up && o2 + 1 == 2;
  if (d0) join_reset(c0);
  if (d1) join_reset(c1);
  if (d2) join_reset(cp);
  strict_release();
  const unsigned to = __shfl(t, 0), tl = __shfl(t, 1), tb = __shfl(t, 2);
  if (f && d0) ring_put(W.out, to + __popcll(mo & lt), MSG_MAKE(0, p.s, p.n));
  if (leaf0) ring_put(down, tl + __popcll(ml0 & lt), MSG_MAKE(1, p.s, BR ? p.a : p.n));
  if (leaf1) ring_put(down, tl + __popcll(ml0) + __popcll(ml1 & lt), MSG_MAKE(1, p.s, p.b));
  if (br0) ring_put(W.branch, tb + __popcll(mb0 & lt), MSG_MAKE(1, p.s, p.a));
  if (br1) ring_put(W.branch, tb + __popcll(mb0) + __popcll(mb1 & lt), MSG_MAKE(1, p.s, p.b));
  const unsigned long long mp = __ballot(d2);
  if (mp) {
    if (lane == 0) t = ring_reserve(W.branch, __popcll(mp));
    t = __shfl(t, 0);
    if (d2) ring_put(W.branch, t + __popcll(mp & lt), MSG_MAKE(0, p.s, p.par >> 1));
  }
}

// ------------------------------------------------------------ lookup
__device__ __noinline__ void role_tree_lookup(const GQ AmpDev* D, const GQ WorkerDev* W) {
  float* lds = amp_lds;
  const GQ NodeDev& lk = D->node[0];
  const TreeBufs B = tree_bufs(D);
  const WorkerRegs wr = worker_regs(D, W);
  const int E = B.E, Ep = B.Ep, KB = wr.kb, E4 = E >> 2, lk_muf = uni(lk.muf);
  const GQ int* smeta = uni_gq<int>(D->smeta);
  int* left_cnt = (int*)lds;                  // [mak] leaves not yet answered
  int* pend_tok = left_cnt + ((D->mak + 3) & ~3);
  for (int i = threadIdx.x; i < D->mak; i += AMP_THREADS) left_cnt[i] = 0;
  BatchMsg& M = s_M;
  const Ring mine = ring_regs(D, uni(W->ring));
  unsigned head = 0;
  unsigned count = W->wstate[0], tstep = W->wstate[1];
  GQ int* keep = (GQ int*)D->buf[10];
  GQ float* prow = (GQ float*)D->buf[11];
  GQ float* lkP = (GQ float*)lk.P;
  const GQ int* tokens = (const GQ int*)D->data.tok;
  GQ float* probe = uni_gq<float>(D->probe);
  GQ unsigned* probe_n = uni_gq<unsigned>(D->probe_n);
  const unsigned probe_period = uni(D->probe_period), probe_cap = uni(D->probe_cap);
  const int probe_w = uni(D->probe_w);
  for (unsigned k = threadIdx.x; k < count; k += AMP_THREADS) pend_tok[k] = keep[k];
  __syncthreads();
  // Wave 1 takes and decodes the next batch while wave 0 is still publishing the present one (wave 0 keeps what its
  // posts need in registers, so the batch's LDS record is free from the publish barrier on).
  const int wave = threadIdx.x >> 6;
  auto take_batch = [&](int room) {
    const int n = poll_batch(D, mine, head, KB, room, s_codes, &s_n, code_is_b);
    if (n > 0) {
      const int k = threadIdx.x & 63;
      if (k < n) {
        const unsigned code = s_codes[k];
        const int s = MSG_SLOT(code), l = MSG_LOCAL(code);
        const v4i sm = tree_slot(smeta, s);
        M.s[k] = s;
        M.n[k] = l;
        M.seq[k] = (unsigned)sm.x;
        M.a[k] = tokens[sm.w + l];
        M.aux[k] = code_is_b(code);
        if (!code_is_b(code) && l == 0) left_cnt[s] = sm.y;
        // probe: the gradient w.r.t. this leaf's embedding (the leaf cell's backward output) of a sampled instance
        int entry = -1;
        if (probe_period && code_is_b(code) && (unsigned)sm.x % probe_period == 0u) {
          const unsigned e = __hip_atomic_fetch_add(probe_n, 1u, __ATOMIC_RELAXED, AGENT);
          if (e < probe_cap) {
            entry = (int)e;
            GQ int* hdr = (GQ int*)(probe + (long long)e * probe_w);
            hdr[0] = 1;
            hdr[1] = sm.x;
            hdr[2] = l;
            hdr[3] = 0;
          }
        }
        M.par[k] = entry;
      }
      batch_split_and_log(D, wr, M, n, 0);
      // backward message k is the b-th gradient of the batch: remember its token
      const bool isb = k < n && M.aux[k] != 0;
      const unsigned long long mb = __ballot(isb);
      if (isb) {
        const int b = __popcll(mb & ((1ull << k) - 1ull));
        M.b[k] = b;
        pend_tok[count + b] = M.a[k];
      }
    }
  };
  if (wave == 1) take_batch(lk_muf - (int)count);
  lds_barrier();
  for (;;) {
    const int n = s_n;
    if (n == 0) break;
    head += n;
    const int nB = M.nB;
    if ((E & 3) == 0) {
      // forward: table row -> xin; backward: sum of the leaf tiles' partials -> pending gradient row
      for (int idx = threadIdx.x; idx < n * E4; idx += AMP_THREADS) {
        const int k = idx / E4, c = (idx - k * E4) << 2;
        if (!M.aux[k]) {
          *(GQ v4f*)(B.xin + B.leaf(M.s[k], M.n[k]) * Ep + c) = *(const GQ v4f*)(lkP + (long long)M.a[k] * E + c);
        } else {
          const GQ float* gx = B.gx + B.leaf(M.s[k], M.n[k]) * B.TL * Ep + c;
          v4f a = {0.f, 0.f, 0.f, 0.f};
          for (int t0 = 0; t0 < B.TL; t0 += 16) {   // sixteen parts in flight at a time, added in tile order
            v4f p[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) p[u] = *(const GQ v4f*)(gx + (t0 + u < B.TL ? t0 + u : B.TL - 1) * Ep);
#pragma unroll
            for (int u = 0; u < 16; ++u)
              if (t0 + u < B.TL) a += p[u];
          }
          *(GQ v4f*)(prow + (long long)(count + M.b[k]) * E + c) = a;
          if (M.par[k] >= 0) *(GQ v4f*)(probe + (long long)M.par[k] * probe_w + 4 + c) = a;
        }
      }
    } else {
      for (int idx = threadIdx.x; idx < n * E; idx += AMP_THREADS) {
        const int k = idx / E, c = idx - k * E;
        if (!M.aux[k]) {
          B.xin[B.leaf(M.s[k], M.n[k]) * Ep + c] = lkP[(long long)M.a[k] * E + c];
        } else {
          const GQ float* gx = B.gx + B.leaf(M.s[k], M.n[k]) * B.TL * Ep + c;
          float a = 0.f;
          for (int t = 0; t < B.TL; ++t) a += gx[t * Ep];
          prow[(long long)(count + M.b[k]) * E + c] = a;
          if (M.par[k] >= 0) probe[(long long)M.par[k] * probe_w + 4 + c] = a;
        }
      }
    }
    // what lane k of wave 0 needs of message k for its post, before the batch's record is given up
    int js = 0, jn = 0, jaux = 0;
    if (threadIdx.x < 64 && (int)threadIdx.x < n) {
      js = M.s[threadIdx.x];
      jn = M.n[threadIdx.x];
      jaux = M.aux[threadIdx.x];
    }
    publish_barrier();
    if (threadIdx.x < 64) {
      fence_release();
      if ((int)threadIdx.x < n) {
        if (!jaux) {
          ring_post(wr.leaf, MSG_MAKE(0, js, jn));
        } else if (wr.train) {
          if (atomicSub(&left_cnt[js], 1) == 1) ring_post(wr.ctl, MSG_MAKE(1, js, 0));
        }
      }
    }
    count += nB;
    if ((int)count >= lk_muf) {
      // SGD on the touched rows: each waiting gradient row is subtracted from its
      // token's row, in arrival order (rows never touched have a zero gradient)
      tstep++;
      if (threadIdx.x == 0) note_update(D);
      const float sc = lk.lr * (lk.mean ? 1.f / (float)count : 1.f);
      __syncthreads();
      for (int c = threadIdx.x; c < E; c += AMP_THREADS) {
        for (unsigned k0 = 0; k0 < count; k0 += 16) {
          const int kc = count - k0 < 16u ? (int)(count - k0) : 16;
          float w[16], g[16];
#pragma unroll
          for (int k = 0; k < 16; ++k)
            if (k < kc) {
              w[k] = lkP[(long long)pend_tok[k0 + k] * E + c];
              g[k] = prow[(long long)(k0 + k) * E + c];
            }
#pragma unroll
          for (int k = 0; k < 16; ++k)
            if (k < kc) {
              // a token seen earlier in this chunk: continue from that result
              float base = w[k];
#pragma unroll
              for (int j = 0; j < 16; ++j)
                if (j < k && pend_tok[k0 + j] == pend_tok[k0 + k]) base = w[j];
              w[k] = base - sc * g[k];
            }
#pragma unroll
          for (int k = 0; k < 16; ++k)
            if (k < kc) lkP[(long long)pend_tok[k0 + k] * E + c] = w[k];
        }
      }
      count = 0;
      lds_barrier();   // every wave has finished with the token list before wave 1 starts the next one
      // recorded by the wave that records the next batch's events, so that the update comes first
      if (threadIdx.x == 64) log_event(D, W, &s_logn, 0, 2, 0, 0);
    }
    if (wave == 1) take_batch(lk_muf - (int)count);
    lds_barrier();
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    W->wstate[0] = count;
    W->wstate[1] = tstep;
  }
  for (unsigned k = threadIdx.x; k < count; k += AMP_THREADS) keep[k] = pend_tok[k];
}

// ------------------------------------------------------------ matrix-core products of a cell tile
// The products are templates over the tile's shape -- NRBT 16-row blocks and
// NCGT 16-column groups, 0 = known only at run time -- because fixed trip
// counts and strides let the compiler unroll the loops, fold the LDS
// addresses into instruction offsets and keep every operand in registers.
// One wave issues at most one matrix instruction every ~32 clocks and needs
// four or more independent accumulators to get there, so the loops below are
// shaped to give every wave an equal share and several accumulators.
#define TREE_XG 20        // 16-column groups of the input held in registers at once
#define TREE_GU 4         // (16-row block, 64-column block) gradient units per wave

template <int NRBT, int NCGT>
struct TreeShape {
  int NRB, NCG, ldw, ldy;
  __device__ __forceinline__ TreeShape(const Tile& t) {
    NRB = NRBT ? NRBT : t.Rp >> 4;
    NCG = NCGT ? NCGT : amp_round16(t.Cl) >> 4;
    ldw = NCGT ? amp_ldrow(NCGT * 16) : t.ldw;
    ldy = NRBT ? amp_ldrow(NRBT * 16) : amp_ldrow(t.Rp);
  }
};

// Y[j][r] = b[r] + sum_c W[r][c] x_j[c] for the nF forward messages of the batch.
// A 16-message block is shared by 8 / (number of blocks) waves, each taking
// every wpn-th 16-row block of the weights.  A wave fetches its messages'
// inputs from HBM (xbase + M.off0 / off1 for the first / second column
// segment) once, straight into operand registers, and uses them for NJ (up to
// three) row blocks at a time.  Loads are unconditional so that they overlap:
// a column group beyond the input reads a valid address and is replaced by zero.
template <bool BR, int NJ, int NRBT, int NCGT>
__device__ __forceinline__ void tree_fwd_pass(const LDSQ float* Wl, const Tile& t, const LDSQ float* bl, const GQ float* p0,
                                              const GQ float* p1, int r0, int wpn, LDSQ float* yrow) {
  const TreeShape<NRBT, NCGT> sh(t);
  const int lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  constexpr int NA = NJ == 1 ? 4 : 2;   // accumulators per row block
  v4f acc[NJ][NA];
  const LDSQ float* wr[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[j][a] = zero;
    wr[j] = Wl + ((r0 + j * wpn) * 16 + i) * sh.ldw + 4 * q;
  }
  for (int c0 = 0; c0 < sh.NCG; c0 += TREE_XG) {
    v4f x[TREE_XG];
#pragma unroll
    for (int g = 0; g < TREE_XG; ++g) {
      const int lc = (c0 + g) * 16 + 4 * q;
      const bool in = lc < t.Cl;
      const GQ float* p = in ? (BR && lc >= t.segp ? p1 : p0) + (c0 + g) * 16 : p0;
      const v4f v = *(const GQ v4f*)p;
      x[g] = in ? v : zero;
    }
    // all fetches are in flight before the first product waits for one
    asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]),
                      "+v"(x[8]), "+v"(x[9]), "+v"(x[10]), "+v"(x[11]), "+v"(x[12]), "+v"(x[13]), "+v"(x[14]),
                      "+v"(x[15]), "+v"(x[16]), "+v"(x[17]), "+v"(x[18]), "+v"(x[19]));
#pragma unroll
    for (int g = 0; g < TREE_XG; ++g) {
      if (NCGT ? g < NCGT : c0 + g < sh.NCG) {
        v4f w[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) w[j] = *(const LDSQ v4f*)(wr[j] + 16 * (c0 + g));
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          acc[j][0] = MFMA(w[j].x, x[g].x, acc[j][0]);
          acc[j][1] = MFMA(w[j].y, x[g].y, acc[j][1]);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          acc[j][NA == 4 ? 2 : 0] = MFMA(w[j].z, x[g].z, acc[j][NA == 4 ? 2 : 0]);
          acc[j][NA == 4 ? 3 : 1] = MFMA(w[j].w, x[g].w, acc[j][NA == 4 ? 3 : 1]);
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int rb = r0 + j * wpn;
    v4f r = *(const LDSQ v4f*)(bl + rb * 16 + 4 * q);
#pragma unroll
    for (int a = 0; a < NA; ++a) r += acc[j][a];
    *(LDSQ v4f*)(yrow + rb * 16 + 4 * q) = r;
  }
}

template <bool BR, int NRBT, int NCGT>
__device__ __forceinline__ void tree_fwd_mfma(const LDSQ float* Wl, const Tile& t, const LDSQ float* bl, const GQ float* xbase,
                                              const BatchMsg& M, int nF, LDSQ float* Y) {
  const TreeShape<NRBT, NCGT> sh(t);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
  const int NBF = (nF + 15) >> 4;
  const int wpn = NBF == 1 ? 8 : NBF == 2 ? 4 : 2;
  // waves w and w + 4 share a SIMD: rotating the row-block offset with the message block evens out the
  // number of row blocks per SIMD when the blocks do not divide evenly among a block's waves
  const int nb = wave / wpn, sub = (wave - nb * wpn + (wpn >> 1) * (nb & 1)) % wpn;
  if (nb >= NBF) return;
  int mi = nb * 16 + i;
  if (mi > nF - 1) mi = nF - 1;   // rows beyond the batch repeat its last message; their results are dropped
  const int m = M.fidx[mi];
  const GQ float* p0 = xbase + M.off0[m] + 4 * q;
  const GQ float* p1 = xbase + M.off1[m] + 4 * q - t.segp;
  LDSQ float* yrow = Y + (nb * 16 + i) * sh.ldy;
  for (int r0 = sub; r0 < sh.NRB; r0 += 3 * wpn) {
    const int left = (sh.NRB - r0 + wpn - 1) / wpn;   // row blocks r0, r0 + wpn, ... still to do
    if (left >= 3)
      tree_fwd_pass<BR, 3, NRBT, NCGT>(Wl, t, bl, p0, p1, r0, wpn, yrow);
    else if (left == 2)
      tree_fwd_pass<BR, 2, NRBT, NCGT>(Wl, t, bl, p0, p1, r0, wpn, yrow);
    else
      tree_fwd_pass<BR, 1, NRBT, NCGT>(Wl, t, bl, p0, p1, r0, wpn, yrow);
  }
}

// dx_j[c] = sum_r W[r][c] delta_j[r] for the nB backward messages; delta rows
// in LDS (Dl, zero beyond the tile's rows); the result goes from the
// accumulators to HBM at obase + M.dst0 / dst1 (+ column inside the
// segment).  Wave item = 16 weight columns, for all NBB message blocks.
template <bool BR, int NBB, int NRBT, int NCGT>
__device__ __forceinline__ void tree_bwd_blocks(const LDSQ float* Wl, const Tile& t, const LDSQ float* Dl, const BatchMsg& M,
                                                int nB, GQ float* obase) {
  const TreeShape<NRBT, NCGT> sh(t);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  constexpr int NA = NBB == 1 ? 4 : 2;
  for (int cb = wave; cb < sh.NCG; cb += AMP_THREADS / 64) {
    const LDSQ float* wp = Wl + (4 * q) * sh.ldw + cb * 16 + i;
    const LDSQ float* dp = Dl + i * sh.ldy + 4 * q;
    v4f acc[NBB][NA];
#pragma unroll
    for (int nb = 0; nb < NBB; ++nb)
#pragma unroll
      for (int a = 0; a < NA; ++a) acc[nb][a] = zero;
#pragma unroll 6
    for (int g = 0; g < sh.NRB; ++g) {
      v4f d[NBB];
#pragma unroll
      for (int nb = 0; nb < NBB; ++nb) d[nb] = *(const LDSQ v4f*)(dp + nb * 16 * sh.ldy + 16 * g);
      const LDSQ float* w = wp + 16 * g * sh.ldw;
      const float a0 = w[0], a1 = w[sh.ldw], a2 = w[2 * sh.ldw], a3 = w[3 * sh.ldw];
#pragma unroll
      for (int nb = 0; nb < NBB; ++nb) {
        acc[nb][0] = MFMA(a0, d[nb].x, acc[nb][0]);
        acc[nb][1] = MFMA(a1, d[nb].y, acc[nb][1]);
      }
#pragma unroll
      for (int nb = 0; nb < NBB; ++nb) {
        acc[nb][NA == 4 ? 2 : 0] = MFMA(a2, d[nb].z, acc[nb][NA == 4 ? 2 : 0]);
        acc[nb][NA == 4 ? 3 : 1] = MFMA(a3, d[nb].w, acc[nb][NA == 4 ? 3 : 1]);
      }
    }
    const int lc = cb * 16 + 4 * q;
#pragma unroll
    for (int nb = 0; nb < NBB; ++nb) {
      const int mi = nb * 16 + i;
      if (mi < nB && lc < t.Cl) {
        const int m = M.bidx[mi];
        GQ float* o = (BR && lc >= t.segp) ? obase + M.dst1[m] + (lc - t.segp) : obase + M.dst0[m] + lc;
        v4f r = acc[nb][0] + acc[nb][1];
        if (NA == 4) r += acc[nb][2] + acc[nb][3];
        *(GQ v4f*)o = r;
      }
    }
  }
}

template <bool BR, int NRBT, int NCGT>
__device__ __forceinline__ void tree_bwd_mfma(const LDSQ float* Wl, const Tile& t, const LDSQ float* Dl, const BatchMsg& M,
                                              int nB, GQ float* obase) {
  const int NBB = (nB + 15) >> 4;
  if (NBB == 1)
    tree_bwd_blocks<BR, 1, NRBT, NCGT>(Wl, t, Dl, M, nB, obase);
  else if (NBB == 2)
    tree_bwd_blocks<BR, 2, NRBT, NCGT>(Wl, t, Dl, M, nB, obase);
  else if (NBB == 3)
    tree_bwd_blocks<BR, 3, NRBT, NCGT>(Wl, t, Dl, M, nB, obase);
  else
    tree_bwd_blocks<BR, 4, NRBT, NCGT>(Wl, t, Dl, M, nB, obase);
}

// Momentum / Adam slots of units U0 .. U0 + US - 1 of a wave, fetched from HBM together: element (v, e) of a unit lies at gi
// (-1 = padding) of the node's slot arrays.
template <int US>
struct TreeSlots {
  int gi[US][4][4];
  float m[US][4][4], v[US][4][4];
};
template <int US>
__device__ __forceinline__ void tree_slots_fetch(TreeSlots<US>& sl, int u0, int NU, int NRB, int cols, int kind, const GQ float* Mq,
                                                 const GQ float* Vq, const LDSQ int* rowmap, const LDSQ int* colmap) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
#pragma unroll
  for (int u = 0; u < US; ++u) {
    const int id = wave + 8 * (u0 + u), cm = id / NRB, rb = id - cm * NRB;
    if (id < NU) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int nc = colmap[cm * 64 + 4 * i + v];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int nr = rowmap[rb * 16 + 4 * q + e];
          sl.gi[u][v][e] = (nr >= 0 && nc >= 0) ? nr * cols + nc : -1;
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int at = sl.gi[u][v][e] >= 0 ? sl.gi[u][v][e] : 0;
          sl.m[u][v][e] = Mq[at];
          sl.v[u][v][e] = kind == 2 ? Vq[at] : 0.f;
        }
    }
  }
}
template <int US, int GU>
__device__ __forceinline__ void tree_slots_step(TreeSlots<US>& sl, int u0, int NU, int NRB, const OptCoef& o, float inv, v4f (&g)[GU][4],
                                                LDSQ float* Wl, int ldw, GQ float* Mq, GQ float* Vq) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
#pragma unroll
  for (int u = 0; u < US; ++u) {
    const int id = wave + 8 * (u0 + u), cm = id / NRB, rb = id - cm * NRB;
    if (u0 + u < GU && id < NU) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int at = sl.gi[u][v][e];
          if (at >= 0) {
            LDSQ float* w = Wl + (rb * 16 + 4 * q + e) * ldw + cm * 64 + 4 * i + v;
            *w = opt_step<true>(o, *w, g[(u0 + u) % GU][v][e] * inv, sl.m[u][v][e], sl.v[u][v][e]);
            Mq[at] = sl.m[u][v][e];
            if (o.kind == 2) Vq[at] = sl.v[u][v][e];
          }
        }
    }
  }
}

// The node's update (Section 3) for one tile, from the `count` pending
// (delta, input) pairs in HBM, entry k at pend + k * stride = [delta (Rp) |
// input in LDS column layout (Cp)]:  G[r][c] = sum_k delta_k[r] x_k[c] in
// arrival order, formed on the matrix cores with the pairs fetched straight
// into operand registers, then the optimizer step on the LDS weights.
// Unit u of a wave is the (16-row block rb, 64-column block cm) with
// rb + NRB * cm = wave + 8 u; its four 16 x 16 tiles take the columns
// cm * 64 + 4 i + v, v = 0..3, so that one 16-byte fetch of an input feeds all
// four.  Lane (i, q) ends up with G[rb*16 + 4q + e][cm*64 + 4i + v] in g[u][v][e].
// gb = the accumulated bias gradient of tile row threadIdx.x; n_grad = the
// number of gradients (messages) behind the count pending rows.
// GU = units per wave: a tile of few units fetches for those alone (a wave without a unit repeats the first one's fetches
// and drops them), and with one or two the next sixteen pairs are on the way while the matrix cores work on the present
// ones.  More units leave no registers for that.
template <int NRBT, int NCGT, int GU>
__device__ __forceinline__ void tree_update_units(LDSQ float* Wl, LDSQ float* bl, const GQ NodeDev& nd, const Tile& t, const GQ float* pend,
                                                  unsigned count, unsigned n_grad, unsigned tstep, const LDSQ int* rowmap,
                                                  const LDSQ int* colmap, float gb) {
  const TreeShape<NRBT, NCGT> sh(t);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
  const int NRB = sh.NRB, Rp = NRB * 16, Cp = sh.NCG * 16, stride = Rp + Cp, CM = (Cp + 63) >> 6, NU = NRB * CM;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  v4f g[GU][4];
  int aoff[GU], xoff[GU];
  bool xin[GU];
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const int id = wave + 8 * u < NU ? wave + 8 * u : 0, cm = id / NRB, rb = id - cm * NRB, lc = cm * 64 + 4 * i;
    aoff[u] = rb * 16 + i;
    xin[u] = lc < Cp;
    xoff[u] = Rp + (xin[u] ? lc : 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) g[u][v] = zero;
  }
  // One unit: the optimizer's slots arrive while the gradient is formed (an update every few gradients is a chain
  // of round trips); more units leave the registers to the gradient.
  constexpr bool EARLY = GU == 1;
  constexpr int US = EARLY ? 1 : 2;
  const int kind = uni(s_opt.o.kind);
  GQ float* Mq = uni_gq<float>(s_opt.M);
  GQ float* Vq = uni_gq<float>(s_opt.V);
  TreeSlots<US> sl;
  float bm = 0.f, bv = 0.f;
  const bool bias = (int)threadIdx.x < t.R && nd.has_bias;
  int bat = 0;
  if (kind != 0) {
    if (bias) {
      bat = nd.rows * t.C + rowmap[threadIdx.x];
      bm = Mq[bat];
      if (kind == 2) bv = Vq[bat];
    }
    if (EARLY) tree_slots_fetch<US>(sl, 0, NU, NRB, t.C, kind, Mq, Vq, rowmap, colmap);
  }
  constexpr int NH = 4;
  // NH groups of four pending pairs, all fetches in flight together
  auto fetch = [&](unsigned k0, float (&a)[NH][GU], v4f (&x)[NH][GU]) {
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const unsigned k = k0 + 4 * h + q;
      const GQ float* e = pend + (long long)(k < count ? k : count - 1) * stride;
#pragma unroll
      for (int u = 0; u < GU; ++u) {
        a[h][u] = e[aoff[u]];
        x[h][u] = *(const GQ v4f*)(e + xoff[u]);
      }
    }
  };
  auto work = [&](unsigned k0, float (&a)[NH][GU], v4f (&x)[NH][GU]) {
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const bool kin = k0 + 4 * h + q < count;
#pragma unroll
      for (int u = 0; u < GU; ++u)
        if (wave + 8 * u < NU) {
          const float av = kin ? a[h][u] : 0.f;
          const v4f xv = xin[u] ? x[h][u] : zero;
          g[u][0] = MFMA(av, xv.x, g[u][0]);
          g[u][1] = MFMA(av, xv.y, g[u][1]);
          g[u][2] = MFMA(av, xv.z, g[u][2]);
          g[u][3] = MFMA(av, xv.w, g[u][3]);
        }
    }
  };
  float a0[NH][GU];
  v4f x0[NH][GU];
  if (GU > 2) {
    for (unsigned k0 = 0; k0 < count; k0 += 4 * NH) {
      fetch(k0, a0, x0);
      asm volatile("" ::: "memory");
      work(k0, a0, x0);
    }
  } else {
    float a1[NH][GU];
    v4f x1[NH][GU];
    if (count > 0) fetch(0, a0, x0);
    for (unsigned k0 = 0; k0 < count; k0 += 8 * NH) {
      if (k0 + 4 * NH < count) fetch(k0 + 4 * NH, a1, x1);
      asm volatile("" ::: "memory");   // the fetches are issued before the products below start
      work(k0, a0, x0);
      if (k0 + 4 * NH >= count) break;
      if (k0 + 8 * NH < count) fetch(k0 + 8 * NH, a0, x0);
      asm volatile("" ::: "memory");
      work(k0 + 4 * NH, a1, x1);
    }
  }
  const OptCoef o = held_opt(tstep);
  const float inv = uni(s_opt.mean) ? 1.f / (float)n_grad : 1.f;
  // optimizer step from the accumulators.  Plain SGD needs no per-element slots: padding rows and columns
  // have a zero gradient (their delta / input entries are zero), so whole 16-byte groups are updated.
  if (kind == 0) {
    const float sc = o.lr * inv;
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      const int id = wave + 8 * u, cm = id / NRB, rb = id - cm * NRB, lc = cm * 64 + 4 * i;
      if (id < NU && lc < Cp) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          LDSQ v4f* wp = (LDSQ v4f*)(Wl + (rb * 16 + 4 * q + e) * sh.ldw + lc);
          const v4f gv = {g[u][0][e], g[u][1][e], g[u][2][e], g[u][3][e]};
          *wp = *wp - sc * gv;
        }
      }
    }
  } else if (EARLY) {
    tree_slots_step<US, GU>(sl, 0, NU, NRB, o, inv, g, Wl, sh.ldw, Mq, Vq);
  } else {
#pragma unroll
    for (int u0 = 0; u0 < GU; u0 += US) {
      tree_slots_fetch<US>(sl, u0, NU, NRB, t.C, kind, Mq, Vq, rowmap, colmap);
      asm volatile("" ::: "memory");   // every fetch is issued before the first store
      tree_slots_step<US, GU>(sl, u0, NU, NRB, o, inv, g, Wl, sh.ldw, Mq, Vq);
    }
  }
  if (bias) {
    bl[threadIdx.x] = opt_step<true>(o, bl[threadIdx.x], gb * inv, bm, bv);
    if (kind != 0) Mq[bat] = bm;
    if (kind == 2) Vq[bat] = bv;
  }
}

template <int NRBT, int NCGT>
__device__ __noinline__ void tree_update_from_pend(LDSQ float* Wl, LDSQ float* bl, const GQ NodeDev* ndp, Tile t,
                                                   const GQ float* pend, unsigned count, unsigned n_grad, unsigned tstep,
                                                   const LDSQ int* rowmap, const LDSQ int* colmap, float gb) {
  if (NRBT) {
    constexpr int GU = NRBT ? (NRBT * ((NCGT * 16 + 63) >> 6) + 7) >> 3 : 1;
    tree_update_units<NRBT, NCGT, GU>(Wl, bl, *ndp, t, pend, count, n_grad, tstep, rowmap, colmap, gb);
  } else {
    const int units = (t.Rp >> 4) * ((amp_round16(t.Cl) + 63) >> 6);
    if (units <= 8)
      tree_update_units<0, 0, 1>(Wl, bl, *ndp, t, pend, count, n_grad, tstep, rowmap, colmap, gb);
    else if (units <= 16)
      tree_update_units<0, 0, 2>(Wl, bl, *ndp, t, pend, count, n_grad, tstep, rowmap, colmap, gb);
    else if (units <= 24)
      tree_update_units<0, 0, 3>(Wl, bl, *ndp, t, pend, count, n_grad, tstep, rowmap, colmap, gb);
    else
      tree_update_units<0, 0, 4>(Wl, bl, *ndp, t, pend, count, n_grad, tstep, rowmap, colmap, gb);
  }
}

// ------------------------------------------------------------ products of a tile whose weights stay in HBM
// For cells too large for the CUs' LDS (hidden size 1024: 12.6 MB and 41.9 MB
// of weights) a tile keeps no copy of its rows: the products read them from
// the node's parameter array (rows x cols, row-major, cols a multiple of 4) in
// HBM / L2 as they go, and the update writes them back in place.  rowoff[lr] =
// (node row of tile row lr) * cols, row 0 for the padding rows of the last
// 16-row block, whose results are dropped or meet a zero delta.

// Y[j][r] = b[r] + sum_c W[r][c] x_j[c], the columns split over the waves: wave w takes the 32-column chunks w, w + 8, ... of
// RG 16-row blocks and all NBF message blocks, weights and inputs straight from memory to operand registers (either is
// fetched once, whole lines), the next chunk's on their way while the matrix cores work on the present one, and no
// barrier until the waves' partial sums meet (through part, nw waves' at a time).  (With the row blocks dealt to the waves, five of them -- hidden 1024 on 64
// tiles -- leave three waves and half of three SIMDs idle: 44 us a batch of 47 instead of 28 us a batch of 37.)
template <bool BR, int NBF, int RG>
__device__ __forceinline__ void tree_fwd_stream_pass(const GQ float* P, const LDSQ int* rowoff, const Tile& t,
                                                     const LDSQ float* bl, const GQ float* xbase, const BatchMsg& M, int nF,
                                                     LDSQ float* Y, int ldy, LDSQ float* part, int nw, int r0) {
  const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
  const int NRB = t.Rp >> 4, nr = NRB - r0 < RG ? NRB - r0 : RG, NCH = (t.Cl + 31) >> 5;
  constexpr int RS = 16 * RG + 4, WS = 16 * NBF * RS;   // floats of a message's / a wave's partial sums
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  const GQ float* wrow[RG];
#pragma unroll
  for (int j = 0; j < RG; ++j) wrow[j] = P + rowoff[(j < nr ? r0 + j : r0) * 16 + i] + 4 * q;
  const GQ float *x0[NBF], *x1[NBF];
#pragma unroll
  for (int nb = 0; nb < NBF; ++nb) {
    const int mi = nb * 16 + i, m = M.fidx[mi < nF ? mi : nF - 1];   // rows beyond the batch repeat its last message; their results are dropped
    x0[nb] = xbase + M.off0[m] + 4 * q;
    x1[nb] = xbase + M.off1[m] + 4 * q - t.segp;
  }
  struct Op {
    v4f w[RG][2], x[NBF][2];
  };
  auto fetch = [&](int ch, Op& o) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c0 = ch * 32 + 16 * h, lc = c0 + 4 * q;
      const bool in = lc < t.Cl;
#pragma unroll
      for (int nb = 0; nb < NBF; ++nb) {
        const v4f v = *(const GQ v4f*)(in ? (BR && lc >= t.segp ? x1[nb] : x0[nb]) + c0 : x0[nb]);
        o.x[nb][h] = in ? v : zero;
      }
#pragma unroll
      for (int j = 0; j < RG; ++j)
        if (j < nr) o.w[j][h] = *(const GQ v4f*)(in ? wrow[j] + c0 : wrow[j]);   // beyond the input: x is zero
    }
  };
  v4f acc[RG][NBF];
#pragma unroll
  for (int j = 0; j < RG; ++j)
#pragma unroll
    for (int nb = 0; nb < NBF; ++nb) acc[j][nb] = zero;
  auto work = [&](const Op& o) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < RG; ++j)
        if (j < nr) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int nb = 0; nb < NBF; ++nb) acc[j][nb] = MFMA(o.w[j][h][e], o.x[nb][h][e], acc[j][nb]);
        }
  };
  Op a, b;
  if (wave < NCH) fetch(wave, a);
  for (int ch = wave; ch < NCH; ch += 16) {
    if (ch + 8 < NCH) fetch(ch + 8, b);
    asm volatile("" ::: "memory");   // the fetches are issued before the products below start
    work(a);
    if (ch + 8 >= NCH) break;
    if (ch + 16 < NCH) fetch(ch + 16, a);
    asm volatile("" ::: "memory");
    work(b);
  }
  // lane (i, q) holds rows 4 q .. 4 q + 3 of message i of a block
  LDSQ float* mine = part + (wave & (nw - 1)) * WS + i * RS + 4 * q;
  for (int s = 8 - nw; s >= 0; s -= nw) {   // waves s .. s + nw - 1 hand theirs to the nw in front of them, the last to everybody
    lds_barrier();                          // part is free
    if (wave >= s && wave < s + nw) {
#pragma unroll
      for (int j = 0; j < RG; ++j)
#pragma unroll
        for (int nb = 0; nb < NBF; ++nb) *(LDSQ v4f*)(mine + nb * 16 * RS + j * 16) = acc[j][nb];
    }
    lds_barrier();
    if (wave < s && wave >= s - nw) {
#pragma unroll
      for (int j = 0; j < RG; ++j)
#pragma unroll
        for (int nb = 0; nb < NBF; ++nb) acc[j][nb] += *(const LDSQ v4f*)(mine + nb * 16 * RS + j * 16);
    }
  }
  const int per = nr * 4;   // groups of four rows
  for (int idx = threadIdx.x; idx < nF * per; idx += AMP_THREADS) {
    const int k = idx / per, r = (idx - k * per) << 2;
    const LDSQ float* p = part + k * RS + r;
    v4f s = *(const LDSQ v4f*)p + *(const LDSQ v4f*)(p + WS);
    if (nw == 4) s += *(const LDSQ v4f*)(p + 2 * WS) + *(const LDSQ v4f*)(p + 3 * WS);
    *(LDSQ v4f*)(Y + k * ldy + r0 * 16 + r) = s + *(const LDSQ v4f*)(bl + r0 * 16 + r);
  }
}

template <bool BR, int NBF>
__device__ __forceinline__ void tree_fwd_stream_blocks(const GQ float* P, const LDSQ int* rowoff, const Tile& t,
                                                       const LDSQ float* bl, const GQ float* xbase, const BatchMsg& M, int nF,
                                                       LDSQ float* Y, int ldy, LDSQ float* part, int nw) {
  constexpr int RG = NBF < 3 ? 6 : NBF == 3 ? 5 : 4;
  for (int r0 = 0; r0 < t.Rp >> 4; r0 += RG) tree_fwd_stream_pass<BR, NBF, RG>(P, rowoff, t, bl, xbase, M, nF, Y, ldy, part, nw, r0);
}

// Ends without a barrier.
template <bool BR>
__device__ __forceinline__ void tree_fwd_stream(const GQ float* P, const LDSQ int* rowoff, const Tile& t, const LDSQ float* bl,
                                                const GQ float* xbase, const BatchMsg& M, int nF, LDSQ float* Y, int ldy,
                                                LDSQ float* part, int nw) {
  const int NBF = (nF + 15) >> 4;
  if (NBF == 1)
    tree_fwd_stream_blocks<BR, 1>(P, rowoff, t, bl, xbase, M, nF, Y, ldy, part, nw);
  else if (NBF == 2)
    tree_fwd_stream_blocks<BR, 2>(P, rowoff, t, bl, xbase, M, nF, Y, ldy, part, nw);
  else if (NBF == 3)
    tree_fwd_stream_blocks<BR, 3>(P, rowoff, t, bl, xbase, M, nF, Y, ldy, part, nw);
  else
    tree_fwd_stream_blocks<BR, 4>(P, rowoff, t, bl, xbase, M, nF, Y, ldy, part, nw);
}

// dx_j[c] = sum_r W[r][c] delta_j[r].  A wave owns every 8th block of 64 weight columns for all NBB message
// blocks.  For a (16-row block, 64-column block) unit lane (i, q) fetches rows 4q .. 4q+3 of the block at columns
// 4i .. 4i+3 -- 16 bytes per fetch, 256 contiguous bytes per row across the 16 lanes -- and component e of those
// fetches is the weight operand of output tile e, whose 16 columns are 4m + e: one fetch feeds four products, and
// a lane ends up with 16 consecutive columns of its message's input gradient.  The rows are walked SR blocks
// at a time with two register buffers, the next stretch in flight while the matrix cores work on the present one.
template <bool BR, int NBB, int SR>
__device__ __forceinline__ void tree_bwd_stream_blocks(const GQ float* P, const LDSQ int* rowoff, const Tile& t,
                                                       const LDSQ float* Dl, int ldd, const BatchMsg& M, int nB, GQ float* obase) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
  const int NRB = t.Rp >> 4, CM = (amp_round16(t.Cl) + 63) >> 6;
  const int NGC = (NRB + SR - 1) / SR;                 // row stretches per column block
  const int ncb = wave < CM ? (CM - wave + 7) >> 3 : 0;           // column blocks of this wave
  const int T = ncb * NGC;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  const LDSQ float* dp = Dl + i * ldd + 4 * q;
  auto afetch = [&](int it, v4f (&a)[SR][4]) {
    const int cb = wave + 8 * (it / NGC), g0 = (it % NGC) * SR;
    const int col = cb * 64 + 4 * i < t.Cl ? cb * 64 + 4 * i : 0;
#pragma unroll
    for (int g = 0; g < SR; ++g) {
      const int gg = g0 + g < NRB ? g0 + g : NRB - 1;
#pragma unroll
      for (int sx = 0; sx < 4; ++sx) a[g][sx] = *(const GQ v4f*)(P + rowoff[gg * 16 + 4 * q + sx] + col);
    }
  };
  v4f acc[NBB][4];
#pragma unroll
  for (int nb = 0; nb < NBB; ++nb)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[nb][e] = zero;
  auto work = [&](int it, v4f (&a)[SR][4]) {
    const int cb = wave + 8 * (it / NGC), gc = it % NGC, g0 = gc * SR;
#pragma unroll
    for (int g = 0; g < SR; ++g)
      if (g0 + g < NRB) {
#pragma unroll
        for (int nb = 0; nb < NBB; ++nb) {
          const v4f d = *(const LDSQ v4f*)(dp + nb * 16 * ldd + 16 * (g0 + g));
#pragma unroll
          for (int sx = 0; sx < 4; ++sx)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[nb][e] = MFMA(a[g][sx][e], d[sx], acc[nb][e]);
        }
      }
    if (gc == NGC - 1) {
#pragma unroll
      for (int nb = 0; nb < NBB; ++nb) {
        const int mi = nb * 16 + i;
        if (mi < nB) {
          const int m = M.bidx[mi];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int lc = cb * 64 + 16 * q + 4 * v;
            if (lc < t.Cl) {
              GQ float* o = (BR && lc >= t.segp) ? obase + M.dst1[m] + (lc - t.segp) : obase + M.dst0[m] + lc;
              *(GQ v4f*)o = (v4f){acc[nb][0][v], acc[nb][1][v], acc[nb][2][v], acc[nb][3][v]};
            }
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[nb][e] = zero;
      }
    }
  };
  v4f a0[SR][4], a1[SR][4];
  if (T > 0) afetch(0, a0);
  for (int it = 0; it < T; it += 2) {
    if (it + 1 < T) afetch(it + 1, a1);
    asm volatile("" ::: "memory");   // the fetches are issued before the products below start
    work(it, a0);
    if (it + 1 >= T) break;
    if (it + 2 < T) afetch(it + 2, a0);
    asm volatile("" ::: "memory");
    work(it + 1, a1);
  }
}

// Row blocks per stretch: four, or three where that leaves less of the last stretch empty (a stretch's fetches are made whole:
// five row blocks as 4 + 1 fetch eight blocks' weights).
template <bool BR, int NBB>
__device__ __forceinline__ void tree_bwd_stream_sr(const GQ float* P, const LDSQ int* rowoff, const Tile& t, const LDSQ float* Dl,
                                                   int ldd, const BatchMsg& M, int nB, GQ float* obase) {
  const int NRB = t.Rp >> 4;
  if ((NRB + 2) / 3 * 3 < (NRB + 3) / 4 * 4)
    tree_bwd_stream_blocks<BR, NBB, 3>(P, rowoff, t, Dl, ldd, M, nB, obase);
  else
    tree_bwd_stream_blocks<BR, NBB, 4>(P, rowoff, t, Dl, ldd, M, nB, obase);
}

template <bool BR>
__device__ __forceinline__ void tree_bwd_stream(const GQ float* P, const LDSQ int* rowoff, const Tile& t, const LDSQ float* Dl,
                                                int ldd, const BatchMsg& M, int nB, GQ float* obase) {
  const int NBB = (nB + 15) >> 4;
  if (NBB == 1)
    tree_bwd_stream_sr<BR, 1>(P, rowoff, t, Dl, ldd, M, nB, obase);
  else if (NBB == 2)
    tree_bwd_stream_sr<BR, 2>(P, rowoff, t, Dl, ldd, M, nB, obase);
  else if (NBB == 3)
    tree_bwd_stream_sr<BR, 3>(P, rowoff, t, Dl, ldd, M, nB, obase);
  else
    tree_bwd_stream_sr<BR, 4>(P, rowoff, t, Dl, ldd, M, nB, obase);
}

// The update of a streamed tile: as tree_update_from_pend, in passes of 8 waves
// x TREE_GU (16-row, 64-column) units, each pass re-reading the pending list;
// the optimizer step goes to the parameter array in HBM.
__device__ __noinline__ void tree_update_stream(GQ float* P, LDSQ float* bl, const GQ NodeDev* ndp, Tile t, const GQ float* pend,
                                                unsigned count, unsigned tstep, const LDSQ int* rowmap, float gb) {
  const GQ NodeDev& nd = *ndp;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
  const int NRB = t.Rp >> 4, Rp = t.Rp, Cp = amp_round16(t.Cl), stride = Rp + Cp, CM = (Cp + 63) >> 6, NU = NRB * CM;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  const OptCoef o = opt_coef(nd, tstep);
  const float inv = nd.mean ? 1.f / (float)count : 1.f;
  constexpr int NH = 4;
  for (int u0 = 0; u0 < NU; u0 += 8 * TREE_GU) {
    v4f g[TREE_GU][4];
    int aoff[TREE_GU], xoff[TREE_GU];
    bool xin[TREE_GU];
#pragma unroll
    for (int u = 0; u < TREE_GU; ++u) {
      const int id = u0 + wave + 8 * u < NU ? u0 + wave + 8 * u : 0, cm = id / NRB, rb = id - cm * NRB, lc = cm * 64 + 4 * i;
      aoff[u] = rb * 16 + i;
      xin[u] = lc < Cp;
      xoff[u] = Rp + (xin[u] ? lc : 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) g[u][v] = zero;
    }
    for (unsigned k0 = 0; k0 < count; k0 += 4 * NH) {
      float a[NH][TREE_GU];
      v4f x[NH][TREE_GU];
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const unsigned k = k0 + 4 * h + q;
        const bool kin = k < count;
        const GQ float* e = pend + (long long)(kin ? k : count - 1) * stride;
#pragma unroll
        for (int u = 0; u < TREE_GU; ++u) {
          const float av = e[aoff[u]];
          const v4f xv = *(const GQ v4f*)(e + xoff[u]);
          a[h][u] = kin ? av : 0.f;
          x[h][u] = xin[u] ? xv : zero;
        }
      }
      asm volatile("" : "+v"(x[0][0]), "+v"(x[0][1]), "+v"(x[0][2]), "+v"(x[0][3]), "+v"(x[1][0]), "+v"(x[1][1]), "+v"(x[1][2]),
                        "+v"(x[1][3]), "+v"(x[2][0]), "+v"(x[2][1]), "+v"(x[2][2]), "+v"(x[2][3]), "+v"(x[3][0]), "+v"(x[3][1]),
                        "+v"(x[3][2]), "+v"(x[3][3]));
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int u = 0; u < TREE_GU; ++u) {
          g[u][0] = MFMA(a[h][u], x[h][u].x, g[u][0]);
          g[u][1] = MFMA(a[h][u], x[h][u].y, g[u][1]);
          g[u][2] = MFMA(a[h][u], x[h][u].z, g[u][2]);
          g[u][3] = MFMA(a[h][u], x[h][u].w, g[u][3]);
        }
    }
#pragma unroll
    for (int u = 0; u < TREE_GU; ++u) {
      const int id = u0 + wave + 8 * u, cm = id / NRB, rb = id - cm * NRB, lc = cm * 64 + 4 * i;
      if (id < NU && lc < t.Cl) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int nr = rowmap[rb * 16 + 4 * q + e];
          if (nr >= 0) {
            const long long gi = (long long)nr * t.C + lc;
            GQ v4f* wp = (GQ v4f*)(P + gi);
            v4f wv = *wp;
#pragma unroll
            for (int v = 0; v < 4; ++v) wv[v] = opt_apply<true>(o, wv[v], g[u][v][e] * inv, (GQ float*)nd.M, (GQ float*)nd.V, gi + v);
            *wp = wv;
          }
        }
      }
    }
  }
  if ((int)threadIdx.x < t.R && nd.has_bias) {
    const int r = threadIdx.x;
    bl[r] = opt_apply<true>(o, bl[r], gb * inv, (GQ float*)nd.M, (GQ float*)nd.V, (long long)nd.rows * t.C + rowmap[r]);
  }
}

// ------------------------------------------------------------ leaf / branch cells
// BR = false: rows [i; o; u] over the embedding.
// BR = true : rows [i; f_l; f_r; o; u] over [h_l; h_r].

// One wave takes the next batch from the ring and decodes it into M: row r of a batch = its forward messages, then its
// backward ones, each in ring order; the event record keeps the ring's order.
template <bool BR>
__device__ __forceinline__ void tree_take(const GQ AmpDev* D, const WorkerRegs& wr, const TreeBufs& B, const Ring& mine, unsigned head,
                                          int room, const GQ int* smeta, const GQ int* tnode) {
  BatchMsg& M = s_M;
  const int n = poll_batch(D, mine, head, wr.kb, room, s_codes, &s_n, code_is_b);
  if (n == 0) return;
  const int lane = threadIdx.x & 63;
  const bool in = lane < n, logs = wr.log_cap && wr.tile == 0;
  const unsigned code = s_codes[in ? lane : 0], base = s_logn;
  const bool isb = in && code_is_b(code), fits = base + (unsigned)n <= wr.log_cap;
  const unsigned long long mb = __ballot(isb), mf = __ballot(in && !isb), lt = (1ull << lane) - 1ull;
  const int nF = __popcll(mf);
  if (in) {
    const int s = MSG_SLOT(code), nn = MSG_LOCAL(code), r = isb ? nF + __popcll(mb & lt) : __popcll(mf & lt);
    const v4i sl = tree_slot(smeta, s);
    const v4i tn = tree_node(tnode, sl.z, nn);
    M.s[r] = s;
    M.n[r] = nn;
    M.a[r] = tn.x;
    M.b[r] = tn.y;
    M.par[r] = tn.z;
    M.L[r] = sl.y;
    if (isb)
      M.bidx[r - nF] = r;
    else
      M.fidx[r] = r;
    if (BR) {
      const int na = s * B.NNmax + tn.x, nb = s * B.NNmax + tn.y;
      M.off0[r] = na * 2 * B.Hp;
      M.off1[r] = nb * 2 * B.Hp;
      M.dst0[r] = (na * B.TB + wr.tile) * B.Hp;
      M.dst1[r] = (nb * B.TB + wr.tile) * B.Hp;
    } else {
      const int l = s * B.Lmax + nn;
      M.off0[r] = M.off1[r] = l * B.Ep;
      M.dst0[r] = M.dst1[r] = (l * B.TL + wr.tile) * B.Ep;
    }
    if (logs && fits)
      wr.log[base + lane] = ((unsigned long long)(unsigned)sl.x << 32) | ((unsigned)(isb ? 1 : 0) << 28) | ((unsigned)wr.node << 20) |
                            ((unsigned)nn & 0xfffffu);
  }
  if (lane == 0) {
    M.nF = nF;
    M.nB = n - nF;
    if (logs) {
      if (fits)
        s_logn = base + (unsigned)n;
      else
        raise_abort(D, ABORT_LOG_FULL, blockIdx.x);
    }
  }
}

// What the delta of one (backward message, unit) pair is formed from: the gate values, the output layer's part, NP of the
// parent tiles' parts and the c's.  All of it is fetched before anything is used; a root, without a parent, reads its parts'
// places and drops them.  (Fetched one after the other where each is needed, with a branch for the root, these are five
// round trips: 2.6 us a batch of 46.)
template <bool BR, int NP>
struct TreeDelta {
  float pp[NP], out, dcp, i_, o_, g_, tc, fl, fr, cl, cr;
  __device__ __forceinline__ void fetch(const TreeBufs& B, const BatchMsg& M, int r, int u, const GQ float* xbase) {
    const int H = B.H, Hp = B.Hp;
    const long long nn = B.node32(M.s[r], M.n[r]);
    const GQ float* gt = B.gate + nn * (6 * H) + u;
    const GQ float* gp = B.gpar + nn * (B.TB * Hp) + u;
    if (NP <= 8 || B.TB > 8) {
#pragma unroll
      for (int a = 0; a < NP; ++a) pp[a] = gp[(a < B.TB ? a : B.TB - 1) * Hp];
    } else {
#pragma unroll
      for (int a = 0; a < 8; ++a) pp[a] = gp[(a < B.TB ? a : B.TB - 1) * Hp];
    }
    out = B.gout[nn * H + u];
    dcp = B.gc[nn * H + u];
    i_ = gt[0];
    o_ = gt[3 * H];
    g_ = gt[4 * H];
    tc = gt[5 * H];
    if (BR) {
      fl = gt[H];
      fr = gt[2 * H];
      cl = xbase[M.off0[r] + Hp + u];
      cr = xbase[M.off1[r] + Hp + u];
    }
  }
  // The delta of unit u = u0 + j (tile order [gate][unit]) into its row ds, and the gradient w.r.t. the children's c.
  __device__ __forceinline__ void form(const TreeBufs& B, const BatchMsg& M, int r, int j, int nu, int u, LDSQ float* ds) const {
    const int H = B.H;
    float p = 0.f;
#pragma unroll
    for (int a = 0; a < NP; ++a)
      if (a < B.TB) p += pp[a];   // in tile order
    if (B.TB > NP) {
      const GQ float* gp = B.gpar + B.node(M.s[r], M.n[r]) * B.TB * B.Hp + u;
      for (int q0 = NP; q0 < B.TB; q0 += NP) {
        float more[NP];
#pragma unroll
        for (int a = 0; a < NP; ++a) more[a] = gp[(q0 + a < B.TB ? q0 + a : B.TB - 1) * B.Hp];
#pragma unroll
        for (int a = 0; a < NP; ++a)
          if (q0 + a < B.TB) p += more[a];
      }
    }
    const bool root = M.par[r] < 0;
    const float dh = root ? out : out + p, dc = root ? 0.f : dcp;
    const float dct = dc + dh * o_ * (1.f - tc * tc);
    const float d_o = dh * tc * o_ * (1.f - o_);
    const float d_i = dct * g_ * i_ * (1.f - i_);
    const float d_g = dct * i_ * (1.f - g_ * g_);
    ds[j] = d_i;
    if (BR) {
      ds[nu + j] = dct * cl * fl * (1.f - fl);
      ds[2 * nu + j] = dct * cr * fr * (1.f - fr);
      ds[3 * nu + j] = d_o;
      ds[4 * nu + j] = d_g;
      B.gc[B.node(M.s[r], M.a[r]) * H + u] = dct * fl;
      B.gc[B.node(M.s[r], M.b[r]) * H + u] = dct * fr;
    } else {
      ds[nu + j] = d_o;
      ds[2 * nu + j] = d_g;
    }
  }
};

// Unit u of node nn from its pre-activations (row y of the tile, unit j of nu): state, and (back) what the way back needs -- six
// stores of eight, which an evaluation has no reader for.
template <bool BR>
__device__ __forceinline__ void tree_activate(const TreeBufs& B, long long nn, const LDSQ float* y, int j, int nu, int u, float cl, float cr,
                                              bool back) {
  const int H = B.H, Hp = B.Hp;
  GQ float* hcn = B.hc + nn * 2 * Hp;
  GQ float* gt = B.gate + nn * 6 * H;
  float c_, o_;
  if (BR) {
    const float i_ = sigmoidf_(y[j]), fl = sigmoidf_(y[nu + j]), fr = sigmoidf_(y[2 * nu + j]);
    o_ = sigmoidf_(y[3 * nu + j]);
    const float g_ = tanh_(y[4 * nu + j]);
    c_ = i_ * g_ + fl * cl + fr * cr;
    if (back) {
      gt[u] = i_;
      gt[H + u] = fl;
      gt[2 * H + u] = fr;
      gt[3 * H + u] = o_;
      gt[4 * H + u] = g_;
    }
  } else {
    const float i_ = sigmoidf_(y[j]);
    o_ = sigmoidf_(y[nu + j]);
    const float g_ = tanh_(y[2 * nu + j]);
    c_ = i_ * g_;
    if (back) {
      gt[u] = i_;
      gt[3 * H + u] = o_;
      gt[4 * H + u] = g_;
    }
  }
  const float tc = tanh_(c_);
  if (back) gt[5 * H + u] = tc;
  hcn[u] = o_ * tc;
  hcn[Hp + u] = c_;
}

// All deltas of a batch into the rows from Y on.  Out of line: inlined, its fetches in flight take registers from the streamed
// products, whose loops then reload theirs from scratch (hidden 1024: 91 ms an epoch of 384 trees instead of 83).
// (The buffers' addresses come through LDS, where the role left them: read from the descriptor in HBM they cost 1.5 %.)
__shared__ TreeBufs s_bufs;
template <bool BR>
__device__ __noinline__ void tree_form_deltas(int nB, int nu, int u0, LDSQ float* Y, int ldy) {
  TreeBufs B;
  B.xin = uni_gq<float>((const void*)s_bufs.xin);
  B.hc = uni_gq<float>((const void*)s_bufs.hc);
  B.gate = uni_gq<float>((const void*)s_bufs.gate);
  B.gout = uni_gq<float>((const void*)s_bufs.gout);
  B.gpar = uni_gq<float>((const void*)s_bufs.gpar);
  B.gc = uni_gq<float>((const void*)s_bufs.gc);
  B.H = uni(s_bufs.H);
  B.Hp = uni(s_bufs.Hp);
  B.NNmax = uni(s_bufs.NNmax);
  B.TB = uni(s_bufs.TB);
  const BatchMsg& M = s_M;
  const GQ float* xbase = BR ? B.hc : B.xin;
  for (int i = threadIdx.x; i < nB * nu; i += AMP_THREADS) {
    const int k = i / nu, r = M.bidx[k], u = u0 + i - k * nu;
    TreeDelta<BR, 16> d;
    d.fetch(B, M, r, u, xbase);
    d.form(B, M, r, i - k * nu, nu, u, Y + k * ldy);
  }
}

// The cells role_tree_cell_lds has no room for.  STREAM: the tile's weights stay in HBM (worker aux = 1); otherwise they
// are in LDS, which is left with fewer rows for a batch's inputs than pay (aux = 0).
// NRBT / NCGT: the tile's 16-row blocks / 16-column groups when known at compile time, else 0.
template <bool BR, int NRBT, int NCGT, bool STREAM>
__device__ __noinline__ void role_tree_cell(const GQ AmpDev* D, const GQ WorkerDev* W) {
  float* lds = amp_lds;
  const GQ NodeDev& nd = D->node[W->node];
  const Tile t = make_tile(nd, W);
  const TreeBufs B = tree_bufs(D);
  if (threadIdx.x == 0) s_bufs = B;   // read after the barriers below
  const Pend pd = make_pend(W, t);
  GQ float* pend = (GQ float*)pd.base;
  const WorkerRegs wr = worker_regs(D, W);
  const int R = t.R, H = B.H, Hp = B.Hp, nu = t.nu, u0 = t.u0, KB = wr.kb, nd_muf = uni(nd.muf);
  const GQ int* smeta = uni_gq<int>(D->smeta);
  const GQ int* tnode = uni_gq<int>(D->data.tnode);
  const int ldy = amp_ldrow(R);
  Lds L{lds};
  float* Wg = L.take(STREAM ? 0 : t.Rp * t.ldw);
  float* bg = L.take(t.Rp);
  LDSQ float* Wl = (LDSQ float*)Wg;
  LDSQ float* bl = (LDSQ float*)bg;
  const int yfloats = KB * ldy;
  LDSQ float* Y = (LDSQ float*)L.take(yfloats);   // forward: pre-activations; backward: deltas
  // node row of a tile row / node column of an LDS column (-1 = padding)
  const int CMW = STREAM ? 0 : ((amp_round16(t.Cl) + 63) >> 6) << 6;
  LDSQ int* rowmap = (LDSQ int*)L.take(t.Rp);
  LDSQ int* colmap = (LDSQ int*)L.take(CMW);
  LDSQ int* rowoff = (LDSQ int*)L.take(STREAM ? t.Rp : 0);   // streamed weights: node row * cols
  const int nw = amp_stream_parts(t.Rp, ldy, KB);
  LDSQ float* part = (LDSQ float*)L.take(STREAM ? nw * 64 * 68 : 0);   // streamed weights: the waves' partial sums
  GQ float* ndP = uni_gq<float>(nd.P);
  if (STREAM) {
    for (int i = threadIdx.x; i < t.Rp; i += AMP_THREADS) {
      rowoff[i] = i < R ? t.grow(i) * t.C : 0;
      bl[i] = (i < R && nd.has_bias) ? ndP[(long long)nd.rows * t.C + t.grow(i)] : 0.f;
    }
  } else {
    tile_load(nd, t, Wg, bg);
  }
  for (int i = threadIdx.x; i < yfloats; i += AMP_THREADS) Y[i] = 0.f;
  for (int i = threadIdx.x; i < t.Rp; i += AMP_THREADS) rowmap[i] = i < R ? t.grow(i) : -1;
  for (int i = threadIdx.x; i < CMW; i += AMP_THREADS) colmap[i] = t.ncol(i);
  __syncthreads();
  // bias gradient of tile row threadIdx.x accumulated since the last update (rests in HBM between launches)
  GQ float* ndG = uni_gq<float>(nd.G);
  float accb = ((int)threadIdx.x < R && nd.has_bias) ? ndG[(long long)nd.rows * t.C + t.grow(threadIdx.x)] : 0.f;
  BatchMsg& M = s_M;
  __syncthreads();
  const Ring mine = ring_regs(D, uni(W->ring));
  const GQ float* xbase = BR ? B.hc : B.xin;
  GQ float* obase = BR ? B.gpar : B.gx;
  unsigned head = 0;
  unsigned count = W->wstate[0], tstep = W->wstate[1];
  // Wave 1 takes the next batch from the ring and decodes it while wave 0 is still publishing the present one
  // (wave 0 keeps what its joins need in registers, so the batch's LDS record is free from the publish barrier on).
  const int wave = threadIdx.x >> 6;
  if (wave == 1) tree_take<BR>(D, wr, B, mine, head, nd_muf - (int)count, smeta, tnode);
  lds_barrier();
  for (;;) {
    const int n = s_n;
    if (n == 0) break;
    head += n;
    const int nF = M.nF, nB = M.nB;
    PHASE(0);
    // ---------------- forward messages of the batch
    if (nF > 0) {
      // the children's c of this thread's first (message, unit) pair travel while the product is formed
      float pcl = 0.f, pcr = 0.f;
      if (BR && (int)threadIdx.x < nF * nu) {
        const int k = threadIdx.x / nu, m = M.fidx[k], u = u0 + (int)threadIdx.x - k * nu;
        pcl = xbase[M.off0[m] + Hp + u];
        pcr = xbase[M.off1[m] + Hp + u];
        asm volatile("" ::: "memory");
      }
      if (STREAM)
        tree_fwd_stream<BR>(ndP, rowoff, t, bl, xbase, M, nF, Y, ldy, part, nw);
      else
        tree_fwd_mfma<BR, NRBT, NCGT>(Wl, t, bl, xbase, M, nF, Y);
      lds_barrier();
      PHASE(1);
      for (int i = threadIdx.x; i < nF * nu; i += AMP_THREADS) {
        const int k = i / nu, j = i - k * nu, m = M.fidx[k], u = u0 + j;
        const bool first = i == (int)threadIdx.x;
        const float cl = BR ? (first ? pcl : xbase[M.off0[m] + Hp + u]) : 0.f;
        const float cr = BR ? (first ? pcr : xbase[M.off1[m] + Hp + u]) : 0.f;
        tree_activate<BR>(B, B.node(M.s[m], M.n[m]), Y + k * ldy, j, nu, u, cl, cr, true);   // (a run-time choice costs this worker 0.8 %)
      }
      lds_barrier();
      PHASE(2);
    }
    // ---------------- backward messages of the batch
    if (nB > 0) {
      // deltas (tile order [gate][unit], zero beyond R) take the pre-activations' place
      for (int i = threadIdx.x; i < nB * (ldy - R); i += AMP_THREADS) {
        const int k = i / (ldy - R), r = R + i - k * (ldy - R);
        Y[k * ldy + r] = 0.f;
      }
      tree_form_deltas<BR>(nB, nu, u0, Y, ldy);
      lds_barrier();
      PHASE(3);
      // The (delta, input) pairs join the pending gradients: entry = [delta (Rp) | input in LDS column layout (Cp)].
      // The input part depends on nothing computed here: its first four 16-byte groups per thread are fetched now,
      // travel while the delta parts are stored and the product is formed, and are stored afterwards.
      const int perx = pd.Cp >> 2, totalx = nB * perx;
      v4f xv[4];
      GQ float* xd[4];
      bool xin[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int idx = threadIdx.x + a * AMP_THREADS;
        const int ii = idx < totalx ? idx : totalx - 1;
        const int k = ii / perx, lc = (ii - k * perx) << 2, m = M.bidx[k];
        xin[a] = lc < t.Cl;
        xd[a] = idx < totalx ? pend + (long long)(count + k) * pd.stride + pd.Rp + lc : nullptr;
        xv[a] = *(const GQ v4f*)(xbase + (xin[a] ? ((BR && lc >= t.segp) ? M.off1[m] + lc - t.segp : M.off0[m] + lc) : M.off0[m]));
      }
      asm volatile("" ::: "memory");   // the fetches are issued before the stores below
      {
        const int perd = pd.Rp >> 2, totald = nB * perd;
        for (int idx = threadIdx.x; idx < totald; idx += AMP_THREADS) {
          const int k = idx / perd, j = (idx - k * perd) << 2;
          *(GQ v4f*)(pend + (long long)(count + k) * pd.stride + j) = *(const LDSQ v4f*)(Y + k * ldy + j);   // ldy >= Rp, zero beyond R
        }
      }
      if ((int)threadIdx.x < R) {
        // the reads of eight messages' deltas are issued together; the sum keeps the messages' order
        int k = 0;
        for (; k + 7 < nB; k += 8) {
          float y[8];
#pragma unroll
          for (int a = 0; a < 8; ++a) y[a] = Y[(k + a) * ldy + threadIdx.x];
#pragma unroll
          for (int a = 0; a < 8; ++a) accb += y[a];
        }
        for (; k < nB; ++k) accb += Y[k * ldy + threadIdx.x];
      }
      PHASE(4);
      if (STREAM)
        tree_bwd_stream<BR>(ndP, rowoff, t, Y, ldy, M, nB, obase);
      else
        tree_bwd_mfma<BR, NRBT, NCGT>(Wl, t, Y, M, nB, obase);
#pragma unroll
      for (int a = 0; a < 4; ++a)
        if (xd[a]) *(GQ v4f*)xd[a] = xin[a] ? xv[a] : (v4f){0.f, 0.f, 0.f, 0.f};
      // the rest of the input parts (batches of more than 4 x 512 groups)
      for (int idx = threadIdx.x + 4 * AMP_THREADS; idx < totalx; idx += AMP_THREADS) {
        const int k = idx / perx, lc = (idx - k * perx) << 2, m = M.bidx[k];
        const bool in = lc < t.Cl;
        const v4f xr = *(const GQ v4f*)(xbase + (in ? ((BR && lc >= t.segp) ? M.off1[m] + lc - t.segp : M.off0[m] + lc) : M.off0[m]));
        *(GQ v4f*)(pend + (long long)(count + k) * pd.stride + pd.Rp + lc) = in ? xr : (v4f){0.f, 0.f, 0.f, 0.f};
      }
      PHASE(5);
    }
    // what lane r of wave 0 needs of row r for its joins, before the batch's record is given up
    const int lane = threadIdx.x & 63;
    const TreePost tp = tree_post_of(M, lane < n ? lane : 0, lane < n, lane < nF);
    // every wave's HBM stores have landed before wave 0 publishes the batch
    publish_barrier();
    // ---------------- joins and posts, one lane per message
    if (wave == 0) {
      fence_release();
      tree_publish<BR>(wr, B, tp);
    }
    PHASE(6);
    count += nB;
    if ((int)count >= nd_muf) {
      // the node's own update (Section 3): optimizer step on the LDS weights with the accumulated gradient
      tstep++;
      if (threadIdx.x == 0) note_update(D);
      if (STREAM)
        tree_update_stream(ndP, bl, &nd, t, pend, count, tstep, rowmap, accb);
      else
        tree_update_from_pend<NRBT, NCGT>(Wl, bl, &nd, t, pend, count, count, tstep, rowmap, colmap, accb);
      accb = 0.f;
      count = 0;
      // recorded by the wave that records the next batch's events, so that the update comes first
      if (threadIdx.x == 64) log_event(D, W, &s_logn, wr.node, 2, 0, 0);
    }
    if (wave == 1) tree_take<BR>(D, wr, B, mine, head, nd_muf - (int)count, smeta, tnode);
    lds_barrier();
    PHASE(7);
  }
  if (STREAM) {
    __syncthreads();
    if ((int)threadIdx.x < R && nd.has_bias) ndP[(long long)nd.rows * t.C + t.grow(threadIdx.x)] = bl[threadIdx.x];
  } else {
    tile_store(nd, t, Wg, bg);
  }
  if ((int)threadIdx.x < R && nd.has_bias) ndG[(long long)nd.rows * t.C + t.grow(threadIdx.x)] = accb;
  if (threadIdx.x == 0) {
    W->wstate[0] = count;
    W->wstate[1] = tstep;
  }
}
