// The recurrent cell's worker with its weights in registers and everything a step touches on the CU.
//
// What bounds it: a sequence's steps follow each other, and a worker has only as many messages to batch as there are
// sequences in flight, so a batch is a chain of short phases and its time is their latency.  role_rnn_cell
// (amp_rnn.hip.h) keeps the weights in LDS, which leaves no room for anything else: every step of a sequence is then a
// ring post and a poll, two descriptor fetches behind each other, inputs fetched by all eight waves, and a pending list
// in HBM -- 16.3 us per batch of 16, where this takes 9.5 us (hidden = emb = 128, an update every 16: 4,000 sequences of
// 4 .. 32 tokens in 101 ms instead of 168; with eight copies 8,000 in 45 ms instead of 71).  Here
//   * the weights are in registers twice, wave w = 4 a + b holding the 64 x 64 piece (rows 64 a .., columns 64 b ..)
//     with a row per lane (forward: contraction over columns) and with a column per lane (backward, update);
//   * the products are v_mfma_f32_4x4x1 over 16 blocks: one operand is four messages' values, broadcast to all blocks,
//     the other 64 rows (columns) of the weights.  The batch is padded to multiples of 4 messages, where 16x16x4 pads to
//     16 -- with 16 sequences in flight a batch has about 7 messages of either direction -- and the rate is higher: two waves
//     on a SIMD issue 512 flop every 5 cycles, measured, against 2,048 every 32 for 16x16x4;
//   * the present input rows, the gradients travelling down the loop, the table, its gradient and the pending
//     (delta, input) pairs are in LDS; HBM holds only the history that the backward steps come back for, stored as it
//     arises and fetched behind the forward product;
//   * the loop edge does not leave the CU: a sequence occupies a lane of wave 0 (its place in the batch) from the message
//     that brings it in to the one that takes it out, and the lane carries slot, step, length and next token.  Messages
//     from other workers are looked for, and their slot's facts fetched, while the present batch is computed.
// The worker's weights (padded to 128 x 256), the table, its gradient and min_update_frequency pairs must fit; a
// larger table or threshold leaves the model to role_rnn_cell.
#pragma once

#define RC_KB 16      // sequences in the worker's hands at a time
#define RC_LDX 144    // rows of the previous output: 16 modulo the 64 banks, so that four messages' reads spread
#define RC_LDD 144    // delta rows, the same
#define RC_PS 384     // a pending pair: delta (128), input (256)
#define RC_TB 1088    // a wave's 16 x 68 floats for turning its weights from one layout into the other
#define RC_H 128      // where an input row's second segment starts

// Row stride of the table and its gradient: whole 64-wide pieces, zero beyond the embedding, so that the forward product
// takes its operands straight from a token's row.
__device__ __forceinline__ int rnn_reg_ldt(int E) { return ((E + 63) & ~63) + 16; }

// LDS floats of this worker with room for `pairs` pending pairs.
__device__ __forceinline__ int rnn_reg_floats(int V, int E, int pairs) {
  return 2 * V * rnn_reg_ldt(E) + RC_KB * (RC_LDX + RC_LDD) + 128 + 8 * RC_TB + 128 + pairs * RC_PS;
}
__device__ __forceinline__ int rnn_reg_pairs(const GQ NodeDev& nd, const GQ WorkerDev* W) {
  const int held = (int)W->wstate[0] + 1;   // pairs carried over from the previous launch, and room for one more
  return nd.muf > held ? nd.muf : held;
}
// Far more sequences in flight than this worker's sixteen places, and a small matrix: role_rnn_cell takes up to 64 messages at
// once, and its padding to 16 costs a small product little, while a batch here takes the same time whatever part of the
// 64-wide pieces is used.  Where the two meet, measured over hidden = emb = 16 .. 128, 17 .. 192 in flight and an update every
// 2 .. 48 (time there / time here, plain SGD; n = sequences in flight for each copy):
//   update every 16: hidden 16 at n = 28 1.06, 32 0.95, 48 0.82; hidden 32 at 32 1.00, 40 0.90; hidden 48 at 40 1.02,
//   48 0.98; hidden 64 at 48 1.05, 64 1.02
//   n = 64: hidden 16 at an update every 10 1.02, 12 0.93; hidden 32 at 12 0.98; hidden 48 at 12 1.07, 14 0.98, 16 0.95;
//   hidden 64 at 16 1.02, 24 0.97, 32 0.94 -- and 1.5 .. 1.7 at 4: updates cut the batches there short
//   more than one piece of rows: hidden 72 at n = 48 and every 24 0.99, n = 64 0.90; hidden 80 1.01, 0.90; hidden 96 1.11,
//   0.98; hidden 128 1.50; with optimizer slots 1.04 .. 1.15 at hidden 80
//   evaluation: hidden 16 at n = 24 1.01, 28 0.88; hidden 32 at 28 0.99, 32 0.89; hidden 48 at 33 1.04, 40 0.96; hidden 64
//   at 40 1.07, 48 0.97; hidden 72 at 40 0.99; hidden 80 at 40 1.04, 48 0.92; hidden 96 at 48 1.04, 64 0.92; hidden 112 1.18
//   emb unlike hidden, n = 64: 32 x 128 at every 32 0.96, evaluation 0.89; 64 x 96 1.08, 0.95; 80 x 128 1.00, 1.01
__device__ __forceinline__ bool rnn_many_in_flight(const GQ AmpDev* D, const GQ NodeDev& nd) {
  const int n = D->mak / D->node_replicas, mean = (nd.rows + D->emb) / 2;
  const int side = (nd.rows > mean ? nd.rows : mean) - (nd.rows > 64 ? 24 : 0);
  if (!D->train) return side <= 80 && n >= 16 + side / 2;
  return side <= 64 && n >= 24 + side / 2 && nd.muf >= 10 + side / 8 && (nd.rows <= 64 || nd.opt == 0);
}
__device__ __forceinline__ bool rnn_reg_fits(const GQ AmpDev* D, const GQ WorkerDev* W) {
  const GQ NodeDev& nd = D->node[W->node];
  const int pairs = rnn_reg_pairs(nd, W);
  if (nd.rows > 128 || D->emb > 128 || nd.seg0 != D->emb || pairs > 96 || D->vocab > 4096) return false;
  if (rnn_many_in_flight(D, nd)) return false;
  return rnn_reg_floats(D->vocab, D->emb, pairs) <= AMP_DYN_LDS_BYTES / 4;
}

// acc[e] += A[4 block + e] * B[lane]: A is block ABID's four values, broadcast to all sixteen blocks.
#define MFMA4(a, b, c, abid) __builtin_amdgcn_mfma_f32_4x4x1f32((a), (b), (c), 4, (abid), 0)
#define RC_MFMA_G(j, kk) acc[(kk) & 3] = MFMA4(xv[j], w[16 * (j) + (kk)], acc[(kk) & 3], kk);
#define RC_MFMA16(j)                                                                                                  \
  RC_MFMA_G(j, 0) RC_MFMA_G(j, 1) RC_MFMA_G(j, 2) RC_MFMA_G(j, 3) RC_MFMA_G(j, 4) RC_MFMA_G(j, 5) RC_MFMA_G(j, 6)     \
  RC_MFMA_G(j, 7) RC_MFMA_G(j, 8) RC_MFMA_G(j, 9) RC_MFMA_G(j, 10) RC_MFMA_G(j, 11) RC_MFMA_G(j, 12)                  \
  RC_MFMA_G(j, 13) RC_MFMA_G(j, 14) RC_MFMA_G(j, 15)

// Four messages against the wave's 64 x 64 piece: part of sum_k w[k] x_m[k] for message m = 0..3 and the lane's row
// (column) in component m.  xp = where lane l finds x[message l % 4][l / 4].
__device__ __forceinline__ v4f rnn_reg_dot(const float (&w)[64], const LDSQ float* xp) {
  float xv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) xv[j] = xp[16 * j];
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  v4f acc[4] = {zero, zero, zero, zero};
  RC_MFMA16(0) RC_MFMA16(1) RC_MFMA16(2) RC_MFMA16(3)
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// The row-per-lane copy of the wave's piece from the column-per-lane one, through the wave's own LDS.
__device__ __forceinline__ void rnn_reg_turn(const float (&wb)[64], float (&wf)[64], LDSQ float* tb) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) {
    if ((lane >> 4) == cc) {
#pragma unroll
      for (int g = 0; g < 16; ++g)
        *(LDSQ v4f*)(tb + (lane & 15) * 68 + 4 * g) = (v4f){wb[4 * g], wb[4 * g + 1], wb[4 * g + 2], wb[4 * g + 3]};
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 16; ++j) wf[16 * cc + j] = tb[j * 68 + lane];
    __builtin_amdgcn_wave_barrier();
  }
}

#define RC_UPD_G(g) acc[(g) & 7] = MFMA4(dv, xv, acc[(g) & 7], g);
#define RC_UPD4(g) RC_UPD_G(g) RC_UPD_G(g + 1) RC_UPD_G(g + 2) RC_UPD_G(g + 3)

// G = sum over the pending pairs, in arrival order, for rows 16 Q .. 16 Q + 16 N - 1 of the wave's piece (N = 1 or 2): row
// 16 Q + 4 g + e of the lane's column in acc[(4 Q + g) & 7][e].
template <int Q, int N>
__device__ __forceinline__ void rnn_reg_gradient(v4f (&acc)[8], const LDSQ float* dp, const LDSQ float* xp, int count) {
  // four pairs' values are fetched ahead of the previous four's products
  float dn[4], xn[4];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int k = h < count ? h : 0;
    dn[h] = dp[k * RC_PS];
    xn[h] = xp[k * RC_PS];
  }
  for (int k0 = 0; k0 < count; k0 += 4) {
    float d4[4], x4[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      d4[h] = dn[h];
      x4[h] = xn[h];
      const int k = k0 + 4 + h < count ? k0 + 4 + h : 0;
      dn[h] = dp[k * RC_PS];
      xn[h] = xp[k * RC_PS];
    }
#pragma unroll
    for (int h = 0; h < 4; ++h)
      if (k0 + h < count) {
        const float dv = d4[h], xv = x4[h];
        RC_UPD4(4 * Q)
        if (N == 2) {
          RC_UPD4(((4 * Q + 4) & 15))
        }
      }
  }
}

// Plain SGD on 32 rows of the column-per-lane copy.
template <int Q>
__device__ __forceinline__ void rnn_reg_sgd(float (&wb)[64], const LDSQ float* dp, const LDSQ float* xp, int count, float sc) {
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  v4f acc[8] = {zero, zero, zero, zero, zero, zero, zero, zero};
  rnn_reg_gradient<Q, 2>(acc, dp, xp, count);
#pragma unroll
  for (int j = 0; j < 32; ++j) wb[16 * Q + j] -= sc * acc[j >> 2][j & 3];
}

// Momentum (OPT 1) / Adam (OPT 2).  The slots are in HBM, consecutive lanes = consecutive columns.  They arrive while the
// first gradient is formed, as many rows' together as the registers hold -- all 64 for momentum, 32 for Adam: a fetch
// behind another row's store would wait for that store.
template <int OPT, int R0, int NR>
__device__ __forceinline__ void rnn_reg_fetch(float (&m)[NR], float (&v)[NR], const GQ float* Mq, const GQ float* Vq, int row0, int rows,
                                              int cols, int col) {
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const int at = (row0 + R0 + j < rows ? row0 + R0 + j : rows - 1) * cols + col;
    m[j] = Mq[at];
    if (OPT == 2) v[j] = Vq[at];
  }
}

// One optimizer step on rows 16 Q .. + 15, whose slots are m[J0 ..], v[J0 ..].
template <int OPT, int Q, int J0, int NR>
__device__ __forceinline__ void rnn_reg_step(float (&wb)[64], float (&m)[NR], float (&v)[NR], const LDSQ float* dp, const LDSQ float* xp,
                                             int count, float inv, const OptCoef& o, GQ float* Mq, GQ float* Vq, int row0, int rows,
                                             int cols, int ncol) {
  const int r0 = row0 + 16 * Q;
  if (r0 >= rows) return;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  v4f acc[8] = {zero, zero, zero, zero, zero, zero, zero, zero};
  rnn_reg_gradient<Q, 1>(acc, dp, xp, count);
  if (J0 == 0) {   // every slot is there before the first is stored
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      asm volatile("" : "+v"(m[j]));
      if (OPT == 2) asm volatile("" : "+v"(v[j]));
    }
  }
  if (ncol >= 0) {
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (r0 + j < rows) {
        float none = 0.f;
        wb[16 * Q + j] = opt_step(o, wb[16 * Q + j], acc[(4 * Q + (j >> 2)) & 7][j & 3] * inv, m[J0 + j], OPT == 2 ? v[J0 + j] : none);
        Mq[(r0 + j) * cols + ncol] = m[J0 + j];
        if (OPT == 2) Vq[(r0 + j) * cols + ncol] = v[J0 + j];
      }
  }
}

// A value the compiler may not compute ahead: without this it hoists the addresses and bounds of all 64 rows of rare
// steps out of the worker's loop and spills what the loop itself needs.
__device__ __forceinline__ int rnn_reg_here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

__device__ __forceinline__ int rnn_reg_here_s(int v) {   // the same in a scalar register
  asm volatile("" : "+s"(v));
  return v;
}

__shared__ unsigned s_rc_ctl;   // a request to the worker itself (message code), taken between two batches; 0 = none

// OPT: the node's optimizer.  SYNC: the launch may send synchronisation requests to the cell's copies.  Both are
// compiled apart because the weights leave half of the registers: what a launch does not use would cost it spills.
template <int OPT, bool SYNC>
__device__ __noinline__ void role_rnn_cell_reg(const GQ AmpDev* D, const GQ WorkerDev* W) {
  const int nc = uni(W->node), nl = nc - 1;   // the cell's node and the table's (1 and 0; a copy's own pair)
  const GQ NodeDev& nd = D->node[nc];
  const GQ NodeDev& lk = D->node[nl];
  const Tile t = make_tile(nd, W);
  const RnnBufs B = rnn_bufs(D);
  const Pend pd = make_pend(W, t);
  GQ float* pend = (GQ float*)pd.base;
  const int H = t.R, E = uni(D->emb), V = uni(D->vocab), C = t.C, SP = B.SP;
  const int tid0 = threadIdx.x, lane0 = tid0 & 63, wave = uni(tid0 >> 6), wa = wave >> 2, wc = wave & 3;
  Lds L{amp_lds};
  const int ldt = rnn_reg_ldt(E), NT = V * ldt;
  LDSQ float* Tab = (LDSQ float*)L.take(NT);
  LDSQ float* Gk = (LDSQ float*)L.take(NT);
  LDSQ float* Z = (LDSQ float*)L.take(128);   // the zero state a sequence starts from
  LDSQ float* X = (LDSQ float*)L.take(RC_KB * RC_LDX);
  LDSQ float* Dl = (LDSQ float*)L.take(RC_KB * RC_LDD);   // gradient w.r.t. the hidden state; in a backward step the delta
  LDSQ float* P = (LDSQ float*)L.take(8 * RC_TB);         // parts of the products; between batches the waves' turning space
  LDSQ float* bl = (LDSQ float*)L.take(128);
  LDSQ float* Q = (LDSQ float*)L.take(rnn_reg_pairs(nd, W) * RC_PS);   // pending pairs in arrival order
  GQ float* ndP = uni_gq<float>(nd.P);
  GQ float* lkP = uni_gq<float>(lk.P);
  GQ float* lkG = uni_gq<float>(lk.G);
  const int nd_muf = uni(nd.muf), lk_muf = uni(lk.muf), has_bias = uni(nd.has_bias);
  const float lk_lr = uni(lk.lr);
  const OptCoef ob = opt_base(nd);
  GQ float* ndM = uni_gq<float>(nd.M);
  GQ float* ndV = uni_gq<float>(nd.V);
  const bool bounded = uni(D->admit_bounded) != 0;
  const bool nd_mean = uni(nd.mean) != 0, lk_mean = uni(lk.mean) != 0;
  const Ring mine = ring_regs(D, uni(W->ring)), out = ring_regs(D, 2), ctl = ring_regs(D, 0);
  const GQ int* tokens = uni_gq<int>(D->data.tok);
  const GQ int* smeta = uni_gq<int>(D->smeta);
  unsigned head = 0;
  unsigned count = uni(W->wstate[0]), tstep = uni(W->wstate[1]), lcount = uni(W->wstate[2]), lstep = uni(W->wstate[3]);
  BatchMsg& M = s_M;
  // which node column this lane holds in the column-per-lane copy, and which pieces of the padded matrix hold anything
  const int xcol = 64 * wc + lane0;
  const int ncol = xcol < RC_H ? (xcol < E ? xcol : -1) : (xcol - RC_H < H ? E + xcol - RC_H : -1);
  const int nE = (E + 63) >> 6, nH = (H + 63) >> 6;   // 64-wide pieces of either input segment / of the rows
  const bool on = wa < nH && (wc < 2 ? wc < nE : wc - 2 < nH);
  LDSQ float* tb = P + wave * RC_TB;
  float wf[64], wb[64];
#pragma unroll
  for (int r = 0; r < 64; ++r) {
    const int row = 64 * wa + r;
    wb[r] = row < H && ncol >= 0 ? ndP[row * C + ncol] : 0.f;
  }
  rnn_reg_turn(wb, wf, tb);
  for (int i = tid0; i < NT; i += AMP_THREADS) {
    const int r = i / ldt, c = i - r * ldt;
    Tab[i] = c < E ? lkP[r * E + c] : 0.f;
    Gk[i] = c < E ? lkG[r * E + c] : 0.f;
  }
  if (tid0 < 128) Z[tid0] = 0.f;
  for (int i = tid0; i < RC_KB * RC_LDX; i += AMP_THREADS) X[i] = 0.f;   // beyond the hidden size it stays zero
  for (int i = tid0; i < RC_KB * RC_LDD; i += AMP_THREADS) Dl[i] = 0.f;
  if (tid0 < 128) bl[tid0] = tid0 < H && has_bias ? ndP[H * C + tid0] : 0.f;
  // pairs carried over from the previous launch (HBM layout: [delta (Rp) | input in the node's column layout])
  for (int i = tid0; i < (int)count * RC_PS; i += AMP_THREADS) {
    const int k = i / RC_PS, j = i - k * RC_PS, c = j - 128, seg = c < RC_H ? c : c - RC_H;
    const GQ float* e = pend + (long long)k * pd.stride;
    float v = 0.f;
    if (j < 128)
      v = j < H ? e[j] : 0.f;
    else if (seg < (c < RC_H ? E : H))
      v = e[pd.Rp + (c < RC_H ? seg : t.segp + seg)];
    Q[i] = v;
  }
  if (tid0 == 0) s_rc_ctl = 0;
  __syncthreads();
  // ---- wave 0's lanes: the sequence lane k < RC_KB holds, as its next message stands
  bool have = false, isb = false, fresh = false;
  int s = 0, tt = 0, len = 0, toff = 0, tok = 0, inst = 0;
  unsigned seq = 0;
  int turn = 0;   // the lane whose backward message goes first when an update cuts the batch
  for (;;) {
    // thread indices and what follows from them are computed anew in every batch: cheaper than the spills they cost as
    // loop invariants
    const int tid = rnn_reg_here(threadIdx.x), lane = tid & 63;
    // ---------------- wave 0 fills its free lanes from ring entry `e` (lane j: the entry of ticket head + j); returns
    // whether anything was taken.  The taken lanes' slot facts follow with facts() and their tokens with token().
    bool taken = false;
    auto take = [&](unsigned long long e) -> bool {
      const bool ready = lane < RC_KB && (unsigned)(e >> 32) == head + (unsigned)lane + 1u;
      const unsigned code = (unsigned)e;
      unsigned long long m = __ballot(ready);
      int n = ~m ? __builtin_ctzll(~m) : 64;
      // a request to the worker itself waits for the end of the batch; what stands behind it stays in the ring
      const unsigned long long mc = __ballot(ready && MSG_SLOT(code) == MSG_CTL_SLOT);
      if (mc) {
        const int first = __builtin_ctzll(mc);
        if (first < n) n = first;
        if (n == 0 && first == 0) {
          fence_acquire();
          if (lane == 0) {
            s_rc_ctl = code;
            s_stat[1] += 1ull;
          }
          head += 1u;
          return true;
        }
      }
      const unsigned long long fr = __ballot(lane < RC_KB && !have);
      const int nfree = __popcll(fr);
      if (n > nfree) n = nfree;
      if (n <= 0) return false;
      fence_acquire();
      const int rank = __popcll(fr & ((1ull << lane) - 1ull));
      const unsigned mycode = __shfl(code, rank & 63);
      taken = lane < RC_KB && !have && rank < n;
      if (taken) {
        have = true;
        fresh = true;
        s = MSG_SLOT(mycode);
        tt = MSG_LOCAL(mycode);
        isb = (mycode & MSG_DIR_B) != 0u;
      }
      head += (unsigned)n;
      return true;
    };
    auto probe = [&]() -> unsigned long long {
      return lane < RC_KB ? __hip_atomic_load((GQ unsigned long long*)&mine.ent[(head + (unsigned)lane) & mine.mask], __ATOMIC_RELAXED, AGENT) : 0ull;
    };
    // ---------------- wave 0: wait if it holds nothing, then lay out the batch
    bool post = false;
    unsigned pcode = 0, ticket = 0;
    bool to_out = false;
    if (tid < 64) {
      int nsel = 0;
      if (!s_rc_ctl && !__ballot(have)) {
        const long long t0 = wall_clock64();
        unsigned spins = 0;
        for (;;) {
          if (take(probe())) break;
          int stop = 0;
          if (lane == 0 && (++spins & 7u) == 0u) {
            if (ld_u32(&D->ctl[0]) | ld_u32(&D->ctl[1])) {
              stop = 1;
            } else if (wall_clock64() - t0 > D->watchdog_ticks) {
              raise_abort(D, ABORT_WATCHDOG, blockIdx.x);
              stop = 1;
            }
          }
          stop = __shfl(stop, 0);
          if (stop) {
            // done is raised only when nothing is in flight; a last look avoids losing a message
            if (ld_u32(&D->ctl[0]) == 0u) take(probe());
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
        if (taken) {
          const v4i sm = *(const GQ v4i*)(smeta + 4 * s);   // admission number, length, instance, token offset
          seq = (unsigned)sm.x;
          len = sm.y;
          toff = sm.w;
          tok = tokens[toff + tt];
        }
        taken = false;
        if (lane == 0) s_stat[0] += (unsigned long long)(wall_clock64() - t0);
      }
      if (!s_rc_ctl) {
        // all forward messages; of the backward ones as many as the next update has room for
        int room = nd_muf - (int)count < lk_muf - (int)lcount ? nd_muf - (int)count : lk_muf - (int)lcount;
        if (room < 1) room = 1;
        const unsigned mall = (unsigned)__ballot(have && isb) & 0xffffu;
        const unsigned rot = ((mall >> turn) | (mall << (RC_KB - turn))) & 0xffffu;
        const int ri = (lane - turn) & (RC_KB - 1);
        const bool selb = have && isb && __popc(rot & ((1u << ri) - 1u)) < room;
        const bool sel = have && (!isb || selb);
        const unsigned long long mb = __ballot(selb), mf = __ballot(have && !isb), ms = mb | mf;
        if (__popc(mall) > room) {
          // the next batch starts behind the last one taken
          const unsigned long long lastm = __ballot(selb && __popc(rot & ((1u << ri) - 1u)) == room - 1);
          turn = lastm ? (__builtin_ctzll(lastm) + 1) & (RC_KB - 1) : turn;
        }
        const unsigned long long lt = (1ull << lane) - 1ull;
        nsel = __popcll(ms);
        if (sel) {
          M.s[lane] = s;
          M.n[lane] = tt;
          M.a[lane] = tok;
          M.aux[lane] = fresh;
          if (selb)
            M.bidx[__popcll(mb & lt)] = lane;
          else
            M.fidx[__popcll(mf & lt)] = lane;
          // where the message leads: the next step of its direction, or out of the worker
          post = isb ? tt == 0 : tt + 1 == len;
          to_out = !isb;
          pcode = MSG_MAKE(isb, s, 0);
        }
        if (lane == 0) {
          M.nF = __popcll(mf);
          M.nB = __popcll(mb);
          s_stat[1] += (unsigned long long)nsel;
          s_stat[2] += 1;
#ifdef AMP_PHASE_STATS
          s_stat[3] = wall_clock64();
#endif
        }
        // every message is an event of both hosted nodes: lookup then cell going forward, cell then lookup going back.
        // The forward messages come first: nothing of the batch may stand between the gradient that completes an
        // update and the update.
        if (s_log_cap && nsel) {
          const unsigned base = s_logn;
          GQ unsigned long long* logp = (GQ unsigned long long*)s_log_ptr;
          if (base + 2u * (unsigned)nsel > s_log_cap) {
            if (lane == 0) raise_abort(D, ABORT_LOG_FULL, blockIdx.x);
          } else {
            if (sel) {
              const int k = isb ? __popcll(mf) + __popcll(mb & lt) : __popcll(mf & lt);
              const unsigned long long tail = ((unsigned long long)seq << 32) | ((unsigned)tt & 0xfffffu);
              const unsigned long long dirb = (unsigned long long)(isb ? 1 : 0) << 28;
              logp[base + 2 * k] = tail | dirb | ((unsigned long long)(isb ? nc : nl) << 20);
              logp[base + 2 * k + 1] = tail | dirb | ((unsigned long long)(isb ? nl : nc) << 20);
            }
            if (lane == 0) s_logn = base + 2u * (unsigned)nsel;
          }
        }
        // the lane moves on to its next message
        if (sel) {
          fresh = false;
          if (post)
            have = false;
          else
            tt += isb ? -1 : 1;
        }
      }
      if (lane == 0) {
        s_n = nsel;
        s_ctl[0] = s_rc_ctl;
      }
    }
    lds_barrier();
    const int n = uni(s_n);
    const unsigned ctlcode = uni(s_ctl[0]);   // not s_rc_ctl: wave 0 may already have taken the next request there
    if (SYNC && ctlcode) {
      // A synchronisation round of the cell's copies (Section 5).  First message of a round: publish the parameters as
      // they stand and arrive at the round's counter; the arrival that completes the group sends every copy the
      // second message.  Second message: every copy's publication is there; move to their mean (summed in copy order)
      // and keep what was learned since the own publication; tell the controller.
      const unsigned rl = MSG_LOCAL(ctlcode), rnd = rl >> 1;
      const int NR = uni(D->node_replicas), rep = uni(W->rep);
      GQ float* cS0 = uni_gq<float>(D->node[1].S);
      GQ float* lS0 = uni_gq<float>(D->node[0].S);
      const long long cstr = NR > 1 ? uni_gq<float>(D->node[4].S) - cS0 : 0, lstr = NR > 1 ? uni_gq<float>(D->node[3].S) - lS0 : 0;
      GQ float* cS = cS0 + rep * cstr;
      GQ float* lS = lS0 + rep * lstr;
      if (!(rl & 1u)) {
        const int r0 = rnn_reg_here_s(64 * wa);
#pragma unroll
        for (int r = 0; r < 64; ++r)
          if (r0 + r < H && ncol >= 0) cS[(r0 + r) * C + ncol] = wb[r];
        if (has_bias && tid < H) cS[H * C + tid] = bl[tid];
        for (int i = tid; i < V * E; i += AMP_THREADS) {
          const int r = i / E;
          lS[i] = Tab[r * ldt + i - r * E];
        }
        LOG(nl, 5, rnd, 0);
        LOG(nc, 5, rnd, 0);
        publish_barrier();
        if (tid == 0) {
          fence_release();
          if (join_arrive((GQ int*)&D->ctl[6], NR))
            for (int q = 0; q < NR; ++q) ring_post(D->ring[q == 0 ? 1 : 2 + q], MSG_MAKE(0, MSG_CTL_SLOT, (rnd << 1) | 1u));
        }
      } else {
        const float inv = 1.f / (float)NR;
        const int r0 = rnn_reg_here_s(64 * wa);
#pragma unroll
        for (int r = 0; r < 64; ++r)
          if (r0 + r < H && ncol >= 0) {
            const int gi = (r0 + r) * C + ncol;
            float m = 0.f;
            for (int q = 0; q < NR; ++q) m += cS0[q * cstr + gi];
            wb[r] = m * inv + (wb[r] - cS[gi]);
          }
        if (has_bias && tid < H) {
          const int gi = H * C + tid;
          float m = 0.f;
          for (int q = 0; q < NR; ++q) m += cS0[q * cstr + gi];
          bl[tid] = m * inv + (bl[tid] - cS[gi]);
        }
        for (int i = tid; i < V * E; i += AMP_THREADS) {
          float m = 0.f;
          for (int q = 0; q < NR; ++q) m += lS0[q * lstr + i];
          const int r = i / E;
          LDSQ float* w = Tab + r * ldt + i - r * E;
          *w = m * inv + (*w - lS[i]);
        }
        rnn_reg_turn(wb, wf, tb);
        LOG(nl, 6, rnd, 0);
        LOG(nc, 6, rnd, 0);
        if (tid == 0) ring_post(ctl, MSG_MAKE(1, MSG_CTL_SLOT, rnd));
      }
      __syncthreads();
      if (tid == 0) s_rc_ctl = 0;
      lds_barrier();
      continue;
    }
    if (n == 0) break;
    const int nF = uni(M.nF), nB = uni(M.nB);
    PHASE(0);
    // look for messages of other workers while the batch is computed
    unsigned long long pe = 0;
    if (tid < 64) pe = probe();
    // ---------------- inputs.  Sixteen groups of 32 threads: group g serves the g-th forward message, then the g-th
    // backward one, four columns a thread.
    const int gi = tid >> 5, c4 = (tid & 31) << 2;
    v4f hy = {0.f, 0.f, 0.f, 0.f}, hp = hy, ee = hy, dd = hy;
    int bm = 0, bs = 0, bt = 0, bfresh = 0;
    if (gi < nB) {
      bm = M.bidx[gi];
      bs = M.s[bm];
      bt = M.n[bm];
      bfresh = M.aux[bm];
      if (c4 < SP) {
        hy = *(const GQ v4f*)(B.hs + B.hrow(bs, bt + 1) + c4);
        hp = *(const GQ v4f*)(B.hs + B.hrow(bs, bt) + c4);
        ee = *(const GQ v4f*)(B.es + B.erow(bs, bt) + c4);
        if (bfresh) dd = *(const GQ v4f*)(B.dh + (long long)bs * SP + c4);
      }
    }
    if (nF > 0) {
      // parts over the column pieces: P[piece][message][128 rows]
      if (on)
        for (int m0 = 0; m0 < nF; m0 += 4) {
          int mi = m0 + (lane & 3);
          if (mi > nF - 1) mi = nF - 1;   // rows beyond the batch repeat its last message; their results are dropped
          const int k = M.fidx[mi];
          // lookup: the token's row as the table stands now; a sequence's first step starts from the zero state
          const LDSQ float* x = wc < 2 ? Tab + M.a[k] * ldt + 64 * wc : (M.aux[k] ? Z : X + k * RC_LDX) + 64 * (wc - 2);
          const v4f r = rnn_reg_dot(wf, x + (lane >> 2));
#pragma unroll
          for (int e = 0; e < 4; ++e) P[(wc * RC_KB + m0 + e) * 128 + 64 * wa + lane] = r[e];
        }
    }
    PHASE(1);
    // what arrived meanwhile takes the free places; its slot's facts are on the way during the rest of the batch
    v4i sm = {0, 0, 0, 0};
    if (tid < 64) {
      if (!s_rc_ctl && __ballot(lane < RC_KB && !have)) take(pe);
      if (taken) sm = *(const GQ v4i*)(smeta + 4 * s);
    }
    PHASE(2);
    if (nF > 0) {
      lds_barrier();
      // a wave per message, two units a lane; the token's row is recorded for the backward pass on the way
      for (int g = wave; g < nF; g += AMP_THREADS / 64) {
        const int k = uni(M.fidx[g]), ks = uni(M.s[k]), kt = uni(M.n[k]), c = 2 * lane;
        const v2f ev = *(const LDSQ v2f*)(Tab + uni(M.a[k]) * ldt + (c < ldt ? c : 0));
        v2f z = *(const LDSQ v2f*)(bl + c);
        for (int b = 0; b < nE; ++b) z += *(const LDSQ v2f*)(P + (b * RC_KB + g) * 128 + c);
        for (int b = 2; b < 2 + nH; ++b) z += *(const LDSQ v2f*)(P + (b * RC_KB + g) * 128 + c);
        const v2f y = {tanhf(z.x), tanhf(z.y)};
        LDSQ float* x = X + k * RC_LDX + c;
        GQ float* hr = B.hs + B.hrow(ks, kt + 1) + c;
        GQ float* er = B.es + B.erow(ks, kt) + c;
        if (c + 1 < H) {
          *(LDSQ v2f*)x = y;
          *(GQ v2f*)hr = y;
        } else if (c < H) {
          *x = y.x;
          *hr = y.x;
        }
        if (c + 1 < E)
          *(GQ v2f*)er = ev;
        else if (c < E)
          *er = ev.x;
      }
    }
    PHASE(3);
    if (nB > 0) {
      if (gi < nB) {
        LDSQ float* d = Dl + bm * RC_LDD + c4;
        LDSQ float* q = Q + (count + gi) * RC_PS + c4;
        const v4f g = bfresh ? dd : *(const LDSQ v4f*)d;
        v4f dv, xe, xh;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          dv[j] = c4 + j < H ? g[j] * (1.f - hy[j] * hy[j]) : 0.f;
          xe[j] = c4 + j < E ? ee[j] : 0.f;
          xh[j] = c4 + j < H ? hp[j] : 0.f;
        }
        *(LDSQ v4f*)d = dv;
        // the (delta, input) pair joins the pending gradients
        *(LDSQ v4f*)q = dv;
        *(LDSQ v4f*)(q + 128) = xe;
        *(LDSQ v4f*)(q + 128 + RC_H) = xh;
      }
      lds_barrier();
    }
    // the new messages' facts, every held sequence's next token, and the places in the receivers' rings: all on the way
    // during the product, the rings' entries filled when the batch's stores have landed
    if (tid < 64) {
      if (taken) {
        seq = (unsigned)sm.x;
        len = sm.y;
        toff = sm.w;
      }
      if (have) tok = tokens[toff + tt];
      if (post) ticket = __hip_atomic_fetch_add(to_out ? out.tail : ctl.tail, 1u, __ATOMIC_RELAXED, AGENT);
    }
    PHASE(4);
    if (nB > 0) {
      // parts over the row pieces: P[piece][message][256 input columns]
      if (on)
        for (int m0 = 0; m0 < nB; m0 += 4) {
          int mi = m0 + (lane & 3);
          if (mi > nB - 1) mi = nB - 1;
          const v4f r = rnn_reg_dot(wb, Dl + M.bidx[mi] * RC_LDD + 64 * wa + (lane >> 2));
#pragma unroll
          for (int e = 0; e < 4; ++e) P[(wa * RC_KB + m0 + e) * 256 + xcol] = r[e];
        }
    }
    PHASE(5);
    if (nB > 0) {
      lds_barrier();
      // wave 0 and 1: the lookup's gradient, in arrival order: column c of every row belongs to thread c, no other thread
      // touches it (LDS float additions in place of read and write were slower: 1.9 instead of 1.1 us for this phase)
      if (tid < 128) {
        for (int k0 = 0; k0 < nB; k0 += 8) {   // eight rows' fetches are in flight together
          float d[8];
          int at[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) at[k] = M.bidx[k0 + k < nB ? k0 + k : k0];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int kk = k0 + k < nB ? k0 + k : k0;
            at[k] = M.a[at[k]] * ldt + tid;
            d[k] = P[kk * 256 + tid];
            if (nH > 1) d[k] += P[(RC_KB + kk) * 256 + tid];
          }
          if (tid < E) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
              if (k0 + k < nB) Gk[at[k]] += d[k];
          }
        }
      } else {
        // the other six: what travels down the loop
        for (int k = wave - 2; k < nB; k += AMP_THREADS / 64 - 2) {
          const int c = 2 * lane;
          v2f d = *(const LDSQ v2f*)(P + k * 256 + RC_H + c);
          if (nH > 1) d += *(const LDSQ v2f*)(P + (RC_KB + k) * 256 + RC_H + c);
          *(LDSQ v2f*)(Dl + uni(M.bidx[k]) * RC_LDD + c) = d;   // beyond the hidden size: dropped when the delta is formed
        }
      }
    }
    // every wave's HBM stores have landed before wave 0 publishes what leaves the worker
    publish_barrier();
    if (tid < 64 && __ballot(post)) {
      fence_release();
      if (post) {
        GQ unsigned long long* e = to_out ? out.ent : ctl.ent;
        const unsigned mask = to_out ? out.mask : ctl.mask;
        __hip_atomic_store(&e[ticket & mask], ((unsigned long long)(ticket + 1u) << 32) | pcode, __ATOMIC_RELAXED, AGENT);
      }
    }
    PHASE(6);
    count += (unsigned)nB;
    lcount += (unsigned)nB;
    if ((int)count >= nd_muf) {
      // the cell's own update (Section 3)
      tstep++;
      if (bounded && tid == 0) note_update(D);
      OptCoef o = opt_at(ob, tstep);
      o.kind = OPT;
      const float inv = nd_mean ? 1.f / (float)count : 1.f;
      const LDSQ float* dp = Q + 64 * wa + lane;
      const LDSQ float* xp = Q + 128 + 64 * wc + lane;
      if (on) {
        if (OPT == 0) {
          rnn_reg_sgd<0>(wb, dp, xp, (int)count, o.lr * inv);
          rnn_reg_sgd<2>(wb, dp, xp, (int)count, o.lr * inv);
        } else {
          constexpr int NR = OPT == 1 ? 64 : 32;
          const int r0 = rnn_reg_here_s(64 * wa), col = ncol >= 0 ? ncol : 0;
          float m[NR], v[NR];
          rnn_reg_fetch<OPT, 0>(m, v, ndM, ndV, r0, H, C, col);
          rnn_reg_step<OPT, 0, 0>(wb, m, v, dp, xp, (int)count, inv, o, ndM, ndV, r0, H, C, ncol);
          rnn_reg_step<OPT, 1, 16>(wb, m, v, dp, xp, (int)count, inv, o, ndM, ndV, r0, H, C, ncol);
          if (OPT == 2 && r0 + 32 < H) rnn_reg_fetch<OPT, 32>(m, v, ndM, ndV, r0, H, C, col);
          rnn_reg_step<OPT, 2, 32 % NR>(wb, m, v, dp, xp, (int)count, inv, o, ndM, ndV, r0, H, C, ncol);
          rnn_reg_step<OPT, 3, 48 % NR>(wb, m, v, dp, xp, (int)count, inv, o, ndM, ndV, r0, H, C, ncol);
        }
        // (forming the row-per-lane copy's gradient by a second pass of products instead spilled, and was slower: 115 against
        // 102 ms for 4,000 sequences)
        rnn_reg_turn(wb, wf, tb);
      }
      // the bias, by the last two waves
      const int br = tid - (AMP_THREADS - 128);
      if (has_bias && br >= 0 && br < H) {
        float g = 0.f;
#pragma unroll 8
        for (int k = 0; k < (int)count; ++k) g += Q[k * RC_PS + br];
        bl[br] = opt_apply(o, bl[br], g * inv, ndM, ndV, (long long)H * C + br);
      }
      count = 0;
      LOG(nc, 2, 0, 0);
    }
    if ((int)lcount >= lk_muf) {
      // the lookup's update: plain SGD over the whole (small) table
      lstep++;
      if (bounded && tid == 0) note_update(D);
      const float sc = lk_lr * (lk_mean ? 1.f / (float)lcount : 1.f);
      // by the waves that have no bias to update; the padding's gradient is zero
      for (int i = 4 * tid; tid < AMP_THREADS - 128 && i < NT; i += 4 * (AMP_THREADS - 128)) {
        *(LDSQ v4f*)(Tab + i) -= sc * *(const LDSQ v4f*)(Gk + i);
        *(LDSQ v4f*)(Gk + i) = (v4f){0.f, 0.f, 0.f, 0.f};
      }
      lcount = 0;
      LOG(nl, 2, 0, 0);
    }
    lds_barrier();
    PHASE(7);
  }
  __syncthreads();
  GQ float* endP = uni_gq<float>(nd.P);
  GQ float* endG = uni_gq<float>(nd.G);
  GQ float* tabP = uni_gq<float>(lk.P);
  GQ float* tabG = uni_gq<float>(lk.G);
  GQ float* list = (GQ float*)make_pend(W, t).base;
  const int r0 = rnn_reg_here_s(64 * wa);
#pragma unroll
  for (int r = 0; r < 64; ++r)
    if (r0 + r < H && ncol >= 0) endP[(r0 + r) * C + ncol] = wb[r];
  if (has_bias && tid0 < H) {
    endP[H * C + tid0] = bl[tid0];
    float g = 0.f;   // the bias gradient of the pairs that wait for the next launch
    for (int k = 0; k < (int)count; ++k) g += Q[k * RC_PS + tid0];
    endG[H * C + tid0] = g;
  }
  for (int i = tid0; i < V * E; i += AMP_THREADS) {
    const int r = i / E, at = r * ldt + i - r * E;
    tabP[i] = Tab[at];
    tabG[i] = Gk[at];
  }
  for (int i = tid0; i < (int)count * pd.stride; i += AMP_THREADS) {
    const int k = i / pd.stride, j = i - k * pd.stride, lc = j - pd.Rp;
    const LDSQ float* q = Q + k * RC_PS;
    float v = 0.f;
    if (j < pd.Rp)
      v = j < H ? q[j] : 0.f;
    else if (lc < t.segp)
      v = lc < E ? q[128 + lc] : 0.f;
    else if (lc - t.segp < H)
      v = q[128 + RC_H + lc - t.segp];
    list[i] = v;
  }
  if (tid0 == 0) {
    W->wstate[0] = count;
    W->wstate[1] = tstep;
    W->wstate[2] = lcount;
    W->wstate[3] = lstep;
  }
}
