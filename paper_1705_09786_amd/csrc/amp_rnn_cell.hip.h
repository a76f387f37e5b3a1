// The recurrent cell's worker with its weights in registers and everything a step touches on the CU.
//
// What bounds it: a sequence's steps follow each other, and a worker has only as many messages to batch as there are
// sequences in flight, so a batch is a chain of short phases and its time is their latency.  role_rnn_cell
// (amp_rnn.hip.h) keeps the weights in LDS, which leaves no room for anything else: every step of a sequence is then a
// ring post and a poll, two descriptor fetches behind each other, inputs fetched by all eight waves, and a pending list
// in HBM -- 16.3 us per batch of 16, where this takes 5.8 us per batch of 12.4 (hidden = emb = 128, an update every 16: 4,000
// sequences of 4 .. 32 tokens in 68 ms instead of 168; with eight copies 8,000 in 23 ms instead of 71).  Here
//   * the weights are in registers twice, wave w = 4 a + b holding the 64 x 64 piece (rows 64 a .., columns 64 b ..)
//     with a row per lane (forward: contraction over columns) and with a column per lane (backward, update);
//   * the products are v_mfma_f32_4x4x1 over 16 blocks: one operand is four messages' values, broadcast to all blocks,
//     the other 64 rows (columns) of the weights.  The batch is padded to multiples of 4 messages, where 16x16x4 pads to
//     16 -- with 16 sequences in flight a batch has about 6 messages of either direction -- at the same rate, 512 flop in 8 cycles;
//   * the present input rows, the gradients travelling down the loop, the table, its gradient and the pending
//     (delta, input) pairs are in LDS; HBM holds only the history that the backward steps come back for, stored as it
//     arises and fetched during the products;
//   * the loop edge does not leave the CU: a sequence occupies a lane of wave 0 (its place in the batch) from the message
//     that brings it in to the one that takes it out, and the lane carries slot, step, length and next token.  Messages
//     from other workers are looked for, and their slot's facts fetched, while the present batch is computed;
//   * a batch has two phases and two barriers: the products of both directions (2.1 us, 1.65 of them matrix instructions), then
//     what follows from them (1.3 us) -- waves 1 .. 7 the activations, the deltas of the *next* backward steps, the pairs and
//     the table's gradient, wave 0 the layout of the next batch.  A message that has just come is taken beside one batch, gets
//     its facts, token and delta beside the next, and is served from then on.  What leaves the worker is posted behind the
//     following barrier, for which every wave waits for its stores anyway.  (With a barrier between forward product,
//     activation, deltas, backward product and publication a batch took 5.8 us without its update, now 3.9.)
//   * an update of 16 gradients takes 4.7 us (7.3 before): 2.2 forming the gradient (1.7 of them matrix instructions), 1.1 turning
//     the weights into the second layout (2.0 with a quarter of the lanes storing at a time), the rest bias, table and barrier.
// The worker's weights (padded to 128 x 256), the table, its gradient and min_update_frequency pairs must fit; a
// larger table or threshold leaves the model to role_rnn_cell.
#pragma once

#define RC_KB 16      // sequences in the worker's hands at a time
#define RC_LDX 144    // rows of the previous output: 16 modulo the 64 banks, so that four messages' reads spread
#define RC_LDD 144    // delta rows, the same
#define RC_PP 512     // a message's parts of a product
#define RC_NOPOST 0xffffffffu
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
// Far more sequences in flight than this worker's sixteen places, a small matrix and no gradients: role_rnn_cell takes up to 64
// messages at once, and its padding to 16 costs a small product little, while a batch here takes the same time whatever part
// of the 64-wide pieces is used.  Where the two meet, measured (time there / time here; n = sequences in flight for each copy):
//   evaluation of 1,000 sequences, hidden = emb = 16 at n = 32 1.01, 40 0.86; 24 at 36 1.06, 48 0.88; 32 at 40 1.04, 48 0.94; 40 at
//   48 1.01, 56 0.94; 48 at 48 1.07, 64 0.94; 56 at 56 1.08, 64 1.00, 128 0.94; 64 at 64 1.10, 128 1.06; more than one piece of
//   rows: 72 at 48 1.05, 56 0.98; 80 at 56 1.05, 64 0.97; 88 at 64 1.02, 128 0.98; 96 nowhere
//   emb unlike hidden: 64 x 16 at 36 1.12, 48 0.94; 64 x 32 at 56 1.02, 64 0.95; 16 x 48 at 48 1.03, 56 0.96; 16 x 64 at 128 1.00
//   training, plain SGD, n = 64 and 128: every 32 1.01 .. 1.6, every 48 1.00 .. 1.39, every 80 0.99 .. 1.02 (hidden 16 .. 72)
__device__ __forceinline__ bool rnn_many_in_flight(const GQ AmpDev* D, const GQ NodeDev& nd) {
  const int n = D->mak / D->node_replicas, mean = (nd.rows + D->emb) / 2;
  const int side = (nd.rows > mean ? nd.rows : mean) - (nd.rows > 64 ? 24 : 0);
  return !D->train && side <= 56 && n >= 23 + side * 7 / 10;
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
// (column) in component m.  xv[i] of lane l = x[message l % 4][16 i + l / 4] (rnn_reg_row, from where lane l finds its first).
__device__ __forceinline__ void rnn_reg_row(float (&xv)[4], const LDSQ float* xp) {
#pragma unroll
  for (int j = 0; j < 4; ++j) xv[j] = xp[16 * j];
}
__device__ __forceinline__ v4f rnn_reg_dot(const float (&w)[64], const float (&xv)[4]) {
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  v4f acc[4] = {zero, zero, zero, zero};
  RC_MFMA16(0) RC_MFMA16(1) RC_MFMA16(2) RC_MFMA16(3)
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}
// The parts of the n first of four messages (n the same in every lane).
__device__ __forceinline__ void rnn_reg_parts(const v4f& r, LDSQ float* o, int n) {
  o[0] = r[0];
  if (n > 1) o[RC_PP] = r[1];
  if (n > 2) o[2 * RC_PP] = r[2];
  if (n > 3) o[3 * RC_PP] = r[3];
}

// The row-per-lane copy of the wave's piece from the column-per-lane one: 16 x 16 blocks change places by swaps of half
// waves and rows of lanes, and each is turned through the wave's own LDS, four of them at a time.  A lane's 16 values go
// there as four 16-byte pieces, placed so that the lanes of one store meet all banks.
__device__ __forceinline__ void rnn_reg_turn(const float (&wb)[64], float (&wf)[64], LDSQ float* tb) {
  const int lane = threadIdx.x & 63, i = lane & 15;
  LDSQ float* mine = tb + (lane >> 4) * 272;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    // registers r, r + 16, r + 32, r + 48 of the four rows of lanes: a 4 x 4 turn
    const auto u = __builtin_amdgcn_permlane32_swap(__float_as_uint(wb[r]), __float_as_uint(wb[r + 32]), false, false);
    const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(wb[r + 16]), __float_as_uint(wb[r + 48]), false, false);
    const auto a = __builtin_amdgcn_permlane16_swap(u[0], v[0], false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(u[1], v[1], false, false);
    wf[r] = __uint_as_float(a[0]);
    wf[r + 16] = __uint_as_float(a[1]);
    wf[r + 32] = __uint_as_float(b[0]);
    wf[r + 48] = __uint_as_float(b[1]);
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int p = 0; p < 4; ++p)
      *(LDSQ v4f*)(mine + 16 * i + 4 * (p ^ (i >> 2))) =
          (v4f){wf[16 * g + 4 * p], wf[16 * g + 4 * p + 1], wf[16 * g + 4 * p + 2], wf[16 * g + 4 * p + 3]};
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 16; ++r) wf[16 * g + r] = mine[16 * r + (i ^ (r & 12))];
    __builtin_amdgcn_wave_barrier();
  }
}

#define RC_UPD_G(g) acc[(g) - 4 * Q] = MFMA4(dv, xv, first ? zero : acc[(g) - 4 * Q], g);
#define RC_UPD4(g) RC_UPD_G(g) RC_UPD_G((g) + 1) RC_UPD_G((g) + 2) RC_UPD_G((g) + 3)

// One pair's products; the first pair's need no cleared sums.
template <int Q, int N, bool first>
__device__ __forceinline__ void rnn_reg_outer(v4f (&acc)[4 * N], float dv, float xv) {
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  RC_UPD4(4 * Q)
  if constexpr (N == 4) {
    RC_UPD4(4)
    RC_UPD4(8)
    RC_UPD4(12)
  }
}
// G = sum over the pending pairs (at least one), in arrival order, for rows 16 Q .. 16 Q + 16 N - 1 of the wave's piece (N = 1
// or 4): row 16 Q + 4 g + e of the lane's column in acc[g][e].  Four pairs at a time, a delta of zero for those that are not;
// the next four's values are fetched during their products.
template <int Q, int N>
__device__ __forceinline__ void rnn_reg_gradient(v4f (&acc)[4 * N], const LDSQ float* dp, const LDSQ float* xp, int count) {
  float dn[4], xn[4];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int k = k0 + h < count ? k0 + h : 0;
      dn[h] = dp[k * RC_PS];
      xn[h] = xp[k * RC_PS];
    }
  };
  fetch(0);
  {
    float d4[4], x4[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      d4[h] = h < count ? dn[h] : 0.f;
      x4[h] = xn[h];
    }
    fetch(4);
    rnn_reg_outer<Q, N, true>(acc, d4[0], x4[0]);
#pragma unroll
    for (int h = 1; h < 4; ++h) rnn_reg_outer<Q, N, false>(acc, d4[h], x4[h]);
  }
  for (int k0 = 4; k0 < count; k0 += 4) {
    float d4[4], x4[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      d4[h] = k0 + h < count ? dn[h] : 0.f;
      x4[h] = xn[h];
    }
    fetch(k0 + 4);
#pragma unroll
    for (int h = 0; h < 4; ++h) rnn_reg_outer<Q, N, false>(acc, d4[h], x4[h]);
  }
}

// Plain SGD on the column-per-lane copy.
__device__ __forceinline__ void rnn_reg_sgd(float (&wb)[64], const LDSQ float* dp, const LDSQ float* xp, int count, float sc) {
  v4f acc[16];
  rnn_reg_gradient<0, 4>(acc, dp, xp, count);
#pragma unroll
  for (int j = 0; j < 64; ++j) wb[j] -= sc * acc[j >> 2][j & 3];
}

// Momentum (OPT 1) / Adam (OPT 2) with the slots in LDS: the wave's 64 x 64 of either kind, a lane's four rows together.
template <int OPT, int Q>
__device__ __forceinline__ void rnn_reg_step_lds(float (&wb)[64], LDSQ float* sl, const LDSQ float* dp, const LDSQ float* xp, int count,
                                                 float inv, const OptCoef& o, int rows, bool col) {
  if (16 * Q >= rows) return;
  LDSQ float* s = sl + 4 * (threadIdx.x & 63);
  v4f m[4], v[4], acc[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    m[g] = *(const LDSQ v4f*)(s + 256 * (4 * Q + g));
    if (OPT == 2) v[g] = *(const LDSQ v4f*)(s + 4096 + 256 * (4 * Q + g));
  }
  rnn_reg_gradient<Q, 1>(acc, dp, xp, count);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float mm = m[g][e], vv = OPT == 2 ? v[g][e] : 0.f;
      const float w = opt_step(o, wb[16 * Q + 4 * g + e], acc[g][e] * inv, mm, vv);
      if (col && 16 * Q + 4 * g + e < rows) wb[16 * Q + 4 * g + e] = w;
      m[g][e] = mm;
      if (OPT == 2) v[g][e] = vv;
    }
    *(LDSQ v4f*)(s + 256 * (4 * Q + g)) = m[g];
    if (OPT == 2) *(LDSQ v4f*)(s + 4096 + 256 * (4 * Q + g)) = v[g];
  }
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
  v4f acc[4];
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
        wb[16 * Q + j] = opt_step(o, wb[16 * Q + j], acc[j >> 2][j & 3] * inv, m[J0 + j], OPT == 2 ? v[J0 + j] : none);
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
  // Optimizer slots of the pieces that hold anything, where the LDS has room for them (a small cell: hidden 37 and embedding 50
  // with momentum and an update every 3 gradients 26.1 ms from HBM, 19.2 here, 1,500 sequences)
  const int pieces = ((H + 63) >> 6) * (((E + 63) >> 6) + ((H + 63) >> 6));
  const bool slots = OPT != 0 && rnn_reg_floats(V, E, rnn_reg_pairs(nd, W)) + pieces * OPT * 4096 <= AMP_DYN_LDS_BYTES / 4;
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
  LDSQ float* sl = Q + rnn_reg_pairs(nd, W) * RC_PS + (wa * (nE + nH) + (wc < 2 ? wc : nE + wc - 2)) * (OPT == 0 ? 1 : OPT) * 4096;
  // the bias's slots, a row to every fourth thread
  float bm = 0.f, bv = 0.f;
  if (OPT != 0 && has_bias && tid0 >> 2 < H) {
    bm = ndM[H * C + (tid0 >> 2)];
    if (OPT == 2) bv = ndV[H * C + (tid0 >> 2)];
  }
  if (slots && on)
    for (int r = 0; r < 64; ++r) {
      const bool in = 64 * wa + r < H && ncol >= 0;
      sl[256 * (r >> 2) + 4 * lane0 + (r & 3)] = in ? ndM[(64 * wa + r) * C + ncol] : 0.f;
      if (OPT == 2) sl[4096 + 256 * (r >> 2) + 4 * lane0 + (r & 3)] = in ? ndV[(64 * wa + r) * C + ncol] : 0.f;
    }
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
  __syncthreads();
  // ---- wave 0's lanes: the sequence lane k < RC_KB holds, as its next message stands.  A lane filled in one batch is served
  // from the next one on (elig), when its facts, token and delta are there.
  bool have = false, elig = false, isb = false;
  int s = 0, tt = 0, len = 0, toff = 0, tok = 0;
  unsigned seq = 0;
  unsigned post = RC_NOPOST, ppost = RC_NOPOST;   // what the lane's message of the batch laid out last / of the one before sends
  int turn = 0;   // the lane whose backward message goes first when an update cuts the batch
  int cur = 0;    // which half of the records the present batch is in
  // ---------------- wave 0 fills its free lanes from ring entry `e` (lane j: the entry of ticket head + j); returns
  // whether anything was taken.
  bool taken = false;
  unsigned n_msgs = 0, n_batches = 0;
  unsigned request = 0;   // a request to the worker itself: handled between two batches, what stands behind it stays in the ring
  auto probe = [&](int lane) -> unsigned long long {
    return lane < RC_KB ? __hip_atomic_load((GQ unsigned long long*)&mine.ent[(head + (unsigned)lane) & mine.mask], __ATOMIC_RELAXED, AGENT) : 0ull;
  };
  auto take = [&](int lane, unsigned long long e) -> bool {
    const bool ready = lane < RC_KB && (unsigned)(e >> 32) == head + (unsigned)lane + 1u;
    const unsigned code = (unsigned)e;
    const unsigned m = (unsigned)__ballot(ready);
    if (!(m & 1u)) return false;
    int n = __builtin_ctz(~m);
    const unsigned mc = (unsigned)__ballot(ready && MSG_SLOT(code) == MSG_CTL_SLOT);
    if (mc) {
      const int first = __builtin_ctz(mc);
      if (first < n) n = first;
      if (n == 0) {
        fence_acquire();
        request = uni(code);
        n_msgs++;
        head += 1u;
        return true;
      }
    }
    const unsigned fr = (unsigned)__ballot(lane < RC_KB && !have);
    const int nfree = __popc(fr);
    if (n > nfree) n = nfree;
    if (n <= 0) return false;
    fence_acquire();
    const int rank = __builtin_amdgcn_mbcnt_lo(fr, 0);
    const unsigned mycode = __shfl(code, rank & 63);
    taken = lane < RC_KB && !have && rank < n;
    if (taken) {
      have = true;
      elig = false;
      s = MSG_SLOT(mycode);
      tt = MSG_LOCAL(mycode);
      isb = (mycode & MSG_DIR_B) != 0u;
    }
    head += (unsigned)n;
    return true;
  };
  // ---------------- wave 0 lays out the next batch (records at q): c / lc gradients will have been gathered then, pe = what
  // the ring held a moment ago
  auto lay_out = [&](int lane, int q, int c, int lc, bool busy, unsigned long long pe) {
    ppost = post;
    post = RC_NOPOST;
    taken = false;
    request = 0;
    int stop = 0;
    if (!__ballot(have || ppost != RC_NOPOST) && !busy) {
      // nothing in hand and nothing left to do: wait
      const long long t0 = wall_clock64();
      unsigned spins = 0;
      while (!take(lane, pe)) {
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
          if (ld_u32(&D->ctl[0]) == 0u && take(lane, probe(lane))) stop = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
        pe = probe(lane);
      }
      if (lane == 0) s_stat[0] += (unsigned long long)(wall_clock64() - t0);
      wait_vm();   // the last look's fetch; else it would be waited for wherever its register is used next, in every batch
    } else if (__ballot(lane < RC_KB && !have)) {
      take(lane, pe);
    }
    // all forward messages; of the backward ones as many as the next update has room for
    int room = nd_muf - c < lk_muf - lc ? nd_muf - c : lk_muf - lc;
    if (room < 1) room = 1;
    const bool can = have && elig && !(SYNC && request);
    bool selb = can && isb;
    const bool self = can && !isb;
    const unsigned mall = (unsigned)__ballot(selb);
    if (__popc(mall) > room) {
      const unsigned rot = ((mall >> turn) | (mall << (RC_KB - turn))) & 0xffffu;
      const int ri = (lane - turn) & (RC_KB - 1), before = __popc(rot & ((1u << ri) - 1u));
      // the next batch starts behind the last one taken
      const unsigned lastm = (unsigned)__ballot(selb && before == room - 1);
      selb = selb && before < room;
      turn = (__builtin_ctz(lastm) + 1) & (RC_KB - 1);
    }
    const bool fresh = taken && isb;   // its delta is formed beside this batch
    const unsigned mb = (unsigned)__ballot(selb), mf = (unsigned)__ballot(self), mt = (unsigned)__ballot(fresh);
    const int nF = __popc(mf), nB = __popc(mb);
    if (lane < RC_KB) {
      const int r = __builtin_amdgcn_mbcnt_lo(self ? mf : selb ? mb : mt, 0), j = r + (self ? 0 : selb ? nF : nF + nB);
      if (self || selb || fresh) {
        M.par[q + j] = lane;
        M.s[q + j] = s;
        M.n[q + j] = tt;
        M.a[q + j] = tok;
        M.seq[q + j] = seq;
      }
      // the operands' rows, the r-th message's where lane r % 4 of a product finds it
      const int at = q + 4 * (r & 3) + (r >> 2);
      if (self) {
        M.off0[at] = tok * ldt;
        M.off1[at] = tt ? lane * RC_LDX : -128;   // the zero state lies in front of the rows
        post = tt + 1 == len ? MSG_MAKE(0, s, 0) : RC_NOPOST;
      } else if (selb) {
        M.dst0[at] = lane * RC_LDD;
        post = tt == 0 ? MSG_MAKE(1, s, 0) : RC_NOPOST;
      }
      // the lane moves on to its next message
      if (self || selb) {
        if (post != RC_NOPOST)
          have = false;
        else
          tt += selb ? -1 : 1;
      }
      elig = have;
    }
    if (lane == 0) {
      M.L[q] = nF | nB << 8 | __popc(mt) << 16 | stop << 24;
      M.L[q + 1] = (int)request;
    }
    n_msgs += (unsigned)(nF + nB);
    n_batches += nF + nB > 0;
  };
  // places no message has been laid out in yet are read too, their products dropped
  if (tid0 < 32) M.off0[tid0] = M.off1[tid0] = M.dst0[tid0] = 0;
  if (tid0 < 64) lay_out(lane0, 0, (int)count, (int)lcount, false, 0ull);
  lds_barrier();
  bool landed = false;   // the stores of the batch before have been waited for already
  // The loop begins at a set place: its matrix instructions, 8 bytes each, run slower where they straddle 8-byte boundaries (4,000
  // sequences 68.5 -> 70.4 ms), and where they lie would otherwise follow from the size of other functions.
  asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
  for (;;) {
    // thread indices and what follows from them are computed anew in every batch: cheaper than the spills they cost as
    // loop invariants
    const int tid = rnn_reg_here(threadIdx.x), lane = tid & 63;
    const int q = 16 * cur;
    const int all = uni(M.L[q]), nF = all & 255, nB = all >> 8 & 255, nT = all >> 16 & 255;
    const unsigned ctlcode = SYNC ? (unsigned)uni(M.L[q + 1]) : 0u;
    if (all >> 24) break;
#ifdef AMP_PHASE_STATS
    if (tid == 0) s_stat[3] = wall_clock64();
#endif
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
    }
    // ---------------- the history rows the backward messages come back for: waves 1 .. 7, two messages each (32 threads, columns
    // c4 .. c4 + 3) and wave 1 the last two places' as well
    const int c4 = (tid & 31) << 2;
    int kind[2] = {0, 0}, gk[2] = {0, 0}, gs[2] = {0, 0}, gt[2] = {0, 0};
    v4f hp[2], ee[2];
    if (wave >= 1) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (h == 0 || (wave == 1 && nF + nB + nT > 14)) {
          const int j = (tid >> 5) + (h ? 12 : -2);
          kind[h] = j >= nF + nB + nT ? 0 : j < nF ? 1 : j < nF + nB ? 2 : 3;
          gk[h] = M.par[q + j];
          gs[h] = M.s[q + j];
          gt[h] = M.n[q + j];
          // a step's inputs; of a message that has just come its step's output and the gradient it brings
          if (kind[h] >= 2 && c4 < SP) {
            hp[h] = *(const GQ v4f*)(B.hs + B.hrow(gs[h], kind[h] == 2 ? gt[h] : gt[h] + 1) + c4);
            ee[h] = *(const GQ v4f*)((kind[h] == 2 ? B.es + B.erow(gs[h], gt[h]) : B.dh + (long long)gs[h] * SP) + c4);
          }
        }
    }
    v4i sm = {0, 0, 0, 0};
    unsigned ticket = 0;
    unsigned long long pe = 0;
    if (wave == 0) {
      pe = probe(lane);
      if (have && !taken) tok = tokens[toff + tt];
      if (taken) sm = *(const GQ v4i*)(smeta + 4 * s);   // admission number, length, instance, token offset
      if (ppost != RC_NOPOST && !landed) ticket = __hip_atomic_fetch_add(ppost & MSG_DIR_B ? ctl.tail : out.tail, 1u, __ATOMIC_RELAXED, AGENT);
      // every message is an event of both hosted nodes: lookup then cell going forward, cell then lookup going back.
      // The forward messages come first: nothing of the batch may stand between the gradient that completes an
      // update and the update.
      if (s_log_cap && nF + nB) {
        const unsigned base = s_logn;
        GQ unsigned long long* logp = (GQ unsigned long long*)s_log_ptr;
        if (base + 2u * (unsigned)(nF + nB) > s_log_cap) {
          if (lane == 0) raise_abort(D, ABORT_LOG_FULL, blockIdx.x);
        } else {
          if (lane < nF + nB) {
            const bool bk = lane >= nF;
            const unsigned long long tail = ((unsigned long long)M.seq[q + lane] << 32) | ((unsigned)M.n[q + lane] & 0xfffffu);
            const unsigned long long dirb = (unsigned long long)(bk ? 1 : 0) << 28;
            logp[base + 2 * lane] = tail | dirb | ((unsigned long long)(bk ? nc : nl) << 20);
            logp[base + 2 * lane + 1] = tail | dirb | ((unsigned long long)(bk ? nl : nc) << 20);
          }
          if (lane == 0) s_logn = base + 2u * (unsigned)(nF + nB);
        }
      }
    }
    PHASE(0);
    // ---------------- products of both directions, four messages at a time.  Parts over the column pieces of a forward
    // message (P[message][piece][128 rows]), over the row pieces of a backward one (P[message][piece][256 input columns]).
    if (on) {
      // lookup: the token's row as the table stands now; a sequence's first step starts from the zero state
      const v4i fo = *(const LDSQ v4i*)((wc < 2 ? M.off0 : M.off1) + q + 4 * (lane & 3));
      const v4i bo = *(const LDSQ v4i*)(M.dst0 + q + 4 * (lane & 3));
      const LDSQ float* xf = (wc < 2 ? Tab + 64 * wc : X + 64 * (wc - 2)) + (lane >> 2);
      const LDSQ float* xb = Dl + 64 * wa + (lane >> 2);
      LDSQ float* of = P + 128 * wc + 64 * wa + lane;
      LDSQ float* ob = P + nF * RC_PP + 256 * wa + xcol;
      float xv[4], xn[4], xw[4];
      rnn_reg_row(xv, xf + fo[0]);
      rnn_reg_row(xw, xb + bo[0]);
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (4 * g < nF) {
          if (g < 3) rnn_reg_row(xn, xf + fo[g < 3 ? g + 1 : 3]);   // the next four's values are on the way during the products
          rnn_reg_parts(rnn_reg_dot(wf, xv), of + 4 * g * RC_PP, nF - 4 * g);
#pragma unroll
          for (int i = 0; i < 4; ++i) xv[i] = xn[i];
        }
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (4 * g < nB) {
          if (g < 3) rnn_reg_row(xn, xb + bo[g < 3 ? g + 1 : 3]);
          rnn_reg_parts(rnn_reg_dot(wb, xw), ob + 4 * g * RC_PP, nB - 4 * g);
#pragma unroll
          for (int i = 0; i < 4; ++i) xw[i] = xn[i];
        }
    }
    PHASE(1);
    // every wave's HBM stores of the batch before have landed (and this one's rows are here)
    publish_barrier();
    PHASE(2);
    if (wave == 0) {
      if (!landed && __ballot(ppost != RC_NOPOST)) {
        // what left the worker in the batch before
        publish_fence();
        if (ppost != RC_NOPOST) ring_put(ppost & MSG_DIR_B ? ctl : out, ticket, ppost);
      }
      if (taken) {
        seq = (unsigned)sm.x;
        len = sm.y;
        toff = sm.w;
        tok = tokens[toff + tt];
        asm volatile("" ::"v"(sm.z));   // held until here: reusing it earlier would wait for the fetch
      }
    }
    landed = false;
    // ---------------- results: waves 1 .. 7, while wave 0 lays out the next batch
    if (wave >= 1) {
      const int wide = 64 * (nE > nH ? nE : nH);   // columns that any row of the worker has, in whole pieces
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (h == 0 || (wave == 1 && nF + nB + nT > 14)) {
          const int j = (tid >> 5) + (h ? 12 : -2);
          if (kind[h] == 1 && c4 < wide) {
            const LDSQ float* p = P + j * RC_PP + c4;
            // all four parts' fetches together; a part that does not exist is whatever the space holds
            const v4f z0 = *(const LDSQ v4f*)p, z1 = *(const LDSQ v4f*)(p + 128), z2 = *(const LDSQ v4f*)(p + 256),
                      z3 = *(const LDSQ v4f*)(p + 384), zb = *(const LDSQ v4f*)(bl + c4);
            const v4f ev = *(const LDSQ v4f*)(Tab + M.a[q + j] * ldt + (c4 < ldt ? c4 : 0));
            v4f z = zb + z0, y, e;
            if (nE > 1) z += z1;
            z += z2;
            if (nH > 1) z += z3;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              y[i] = c4 + i < H ? tanh_(z[i]) : 0.f;
              e[i] = c4 + i < E ? ev[i] : 0.f;
            }
            *(LDSQ v4f*)(X + gk[h] * RC_LDX + c4) = y;
            // what the backward pass comes back for: the output and the token's row
            if (c4 < SP) {
              *(GQ v4f*)(B.hs + B.hrow(gs[h], gt[h] + 1) + c4) = y;
              *(GQ v4f*)(B.es + B.erow(gs[h], gt[h]) + c4) = e;
            }
          } else if (kind[h] >= 2 && c4 < wide) {
            LDSQ float* d = Dl + gk[h] * RC_LDD + c4;
            v4f g = ee[h];
            if (kind[h] == 2) {
              // the (delta, input) pair joins the pending gradients, and the step before gets its delta
              LDSQ float* pr = Q + ((int)count + j - nF) * RC_PS + c4;
              v4f xe, xh;
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                xe[i] = c4 + i < E ? ee[h][i] : 0.f;
                xh[i] = c4 + i < H ? hp[h][i] : 0.f;
              }
              *(LDSQ v4f*)pr = *(const LDSQ v4f*)d;
              *(LDSQ v4f*)(pr + 128) = xe;
              *(LDSQ v4f*)(pr + 128 + RC_H) = xh;
              const LDSQ float* p = P + j * RC_PP + RC_H + c4;
              g = *(const LDSQ v4f*)p;
              if (nH > 1) g += *(const LDSQ v4f*)(p + 256);
            }
            v4f dn;
#pragma unroll
            for (int i = 0; i < 4; ++i) dn[i] = c4 + i < H ? g[i] * (1.f - hp[h][i] * hp[h][i]) : 0.f;
            *(LDSQ v4f*)d = dn;
          }
        }
      // the lookup's gradient, in arrival order; each of the seven waves has the tokens of its own
      const int mytok = lane < nB ? M.a[q + nF + lane] : -1;
      unsigned todo = (unsigned)__ballot(mytok >= 0 && mytok % 7 == wave - 1);
      for (; todo; todo &= todo - 1u) {
        const int k = __builtin_ctz(todo);
        LDSQ float* gr = Gk + __builtin_amdgcn_readlane(mytok, k) * ldt + lane;
        const LDSQ float* p = P + (nF + k) * RC_PP + lane;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (h < nE) {
            float d = p[64 * h];
            if (nH > 1) d += p[256 + 64 * h];
            if (lane + 64 * h < E) gr[64 * h] += d;
          }
      }
    }
    PHASE(3);
    count += (unsigned)nB;
    lcount += (unsigned)nB;
    const bool upd_c = (int)count >= nd_muf, upd_l = (int)lcount >= lk_muf;
    if (wave == 0) lay_out(lane, 16 - q, upd_c ? 0 : (int)count, upd_l ? 0 : (int)lcount, upd_c || upd_l, pe);
    cur ^= 1;
    PHASE(4);
    lds_barrier();
    PHASE(2);
    if (!(upd_c || upd_l)) continue;
    // the updates; what leaves the worker is posted behind them
    if (tid < 64 && ppost != RC_NOPOST) ticket = __hip_atomic_fetch_add(ppost & MSG_DIR_B ? ctl.tail : out.tail, 1u, __ATOMIC_RELAXED, AGENT);
    if (upd_c) {
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
          rnn_reg_sgd(wb, dp, xp, (int)count, o.lr * inv);
        } else if (slots) {
          rnn_reg_step_lds<OPT, 0>(wb, sl, dp, xp, (int)count, inv, o, H - 64 * wa, ncol >= 0);
          rnn_reg_step_lds<OPT, 1>(wb, sl, dp, xp, (int)count, inv, o, H - 64 * wa, ncol >= 0);
          rnn_reg_step_lds<OPT, 2>(wb, sl, dp, xp, (int)count, inv, o, H - 64 * wa, ncol >= 0);
          rnn_reg_step_lds<OPT, 3>(wb, sl, dp, xp, (int)count, inv, o, H - 64 * wa, ncol >= 0);
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
        PHASE(5);
        // (forming the row-per-lane copy's gradient by a second pass of products instead spilled, and was slower: 115 against
        // 102 ms for 4,000 sequences)
        rnn_reg_turn(wb, wf, tb);
        PHASE(6);
      }
      // the bias: four threads a row, every fourth pair each
      float gbias = 0.f;
      for (int k = tid & 3; k < (int)count; k += 4) gbias += Q[k * RC_PS + (tid >> 2)];
      gbias += dpp<DPP_XOR1>(gbias);
      gbias += dpp<DPP_XOR2>(gbias);
      if (has_bias && (tid & 3) == 0 && tid >> 2 < H)
        bl[tid >> 2] = opt_step(o, bl[tid >> 2], gbias * inv, bm, bv);
      count = 0;
      LOG(nc, 2, 0, 0);
    }
    if (upd_l) {
      // the lookup's update: plain SGD over the whole (small) table
      lstep++;
      if (bounded && tid == 0) note_update(D);
      const float sc = lk_lr * (lk_mean ? 1.f / (float)lcount : 1.f);
      // the padding's gradient is zero
      for (int i = 4 * tid; i < NT; i += 4 * AMP_THREADS) {
        *(LDSQ v4f*)(Tab + i) -= sc * *(const LDSQ v4f*)(Gk + i);
        *(LDSQ v4f*)(Gk + i) = (v4f){0.f, 0.f, 0.f, 0.f};
      }
      lcount = 0;
      LOG(nl, 2, 0, 0);
    }
    publish_barrier();
    if (tid < 64 && __ballot(ppost != RC_NOPOST)) {
      publish_fence();
      if (ppost != RC_NOPOST) ring_put(ppost & MSG_DIR_B ? ctl : out, ticket, ppost);
    }
    landed = true;
    PHASE(7);
  }
  if (tid0 == 0) {
    s_stat[1] += n_msgs;
    s_stat[2] += n_batches;
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
  if (OPT != 0) {
    GQ float* endM = uni_gq<float>(nd.M);
    GQ float* endV = uni_gq<float>(nd.V);
    if (has_bias && (tid0 & 3) == 0 && tid0 >> 2 < H) {
      endM[H * C + (tid0 >> 2)] = bm;
      if (OPT == 2) endV[H * C + (tid0 >> 2)] = bv;
    }
    if (slots && on && ncol >= 0)
      for (int r = 0; r < 64 && r0 + r < H; ++r) {
        endM[(r0 + r) * C + ncol] = sl[256 * (r >> 2) + 4 * lane0 + (r & 3)];
        if (OPT == 2) endV[(r0 + r) * C + ncol] = sl[4096 + 256 * (r >> 2) + 4 * lane0 + (r & 3)];
      }
  }
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
