// Tree-LSTM output layer: a softmax loss at every tree node, where a forward message turns round (Section 4: the loss
// layer initiates backpropagation).
//
// Every node of every tree visits this one workgroup, so its batch has to be short; it is a chain of round trips around
// little arithmetic.  The batch's h rows go straight to LDS; logits (16 classes x 16 messages, the columns in two
// halves so that more waves share them) and W^T d logits run on the matrix cores; after the hand-over barrier wave 0 joins
// and posts, wave 1 takes the next batch, and only the other six form the gradient and make the update.  Its accumulator
// (n_class x H elements, NG groups of four columns a thread) and the optimizer's slots stay in registers for the life of the launch; between
// launches they rest in HBM.
#pragma once

// Joins and posts of the output layer's batch: one message per lane of the calling wave (all 64 lanes), after a release fence.  A
// training node's part of its gradient is there; the last node of an evaluation instance (fin) retires it.
__device__ __forceinline__ void tree_out_publish(const WorkerRegs& W, const TreeBufs& B, int s, int n, bool grad, bool root, bool is_leaf,
                                                 bool fin) {
  const int lane = threadIdx.x & 63;
  const unsigned long long lt = (1ull << lane) - 1ull;
  GQ int* c = B.cnt + B.node(s, n) * 4 + 2;
  int old = 0;
  if (grad) old = join_add(c);
  const bool done = grad && old + 1 == (root ? 1 : 1 + B.TB), lf = done && is_leaf, br = done && !is_leaf;
  const unsigned long long ml = __ballot(lf), mb = __ballot(br), mc = __ballot(fin);
  const unsigned want = lane == 0 ? __popcll(ml) : lane == 1 ? __popcll(mb) : lane == 2 ? __popcll(mc) : 0u;
  GQ unsigned *const tail_leaf = W.leaf.tail, *const tail_branch = W.branch.tail, *const tail_ctl = W.ctl.tail;
  GQ unsigned* tail = lane == 0 ? tail_leaf : lane == 1 ? tail_branch : tail_ctl;
  unsigned t = 0;
  if (want) t = __hip_atomic_fetch_add(tail, want, __ATOMIC_RELAXED, AGENT);
  if (done) join_reset(c);
  strict_release();
  const unsigned tl = __shfl(t, 0), tb = __shfl(t, 1), tc = __shfl(t, 2);
  if (lf) ring_put(W.leaf, tl + __popcll(ml & lt), MSG_MAKE(1, s, n));
  if (br) ring_put(W.branch, tb + __popcll(mb & lt), MSG_MAKE(1, s, n));
  if (fin) ring_put(W.ctl, tc + __popcll(mc & lt), MSG_MAKE(1, s, 0));
}

// Sums and maxima over groups of GS consecutive lanes (8 .. 64), left in every lane of the group.
template <int GS>
__device__ __forceinline__ float group_sum(float v) {
  v += dpp<DPP_XOR1>(v);
  v += dpp<DPP_XOR2>(v);
  v += dpp<DPP_HALF_MIRROR>(v);
  if (GS > 8) v += dpp<DPP_MIRROR>(v);
  if (GS > 16) v += __shfl_xor(v, 16);
  if (GS > 32) v += __shfl_xor(v, 32);
  return v;
}
__device__ __forceinline__ void take_larger(float& m, int& am, float om, int oa) {
  if (om > m || (om == m && oa < am)) {
    m = om;
    am = oa;
  }
}
template <int GS>
__device__ __forceinline__ void group_argmax(float& m, int& am) {   // the first of equal ones
  take_larger(m, am, dpp<DPP_XOR1>(m), dpp<DPP_XOR1>(am));
  take_larger(m, am, dpp<DPP_XOR2>(m), dpp<DPP_XOR2>(am));
  take_larger(m, am, dpp<DPP_HALF_MIRROR>(m), dpp<DPP_HALF_MIRROR>(am));
  if (GS > 8) take_larger(m, am, dpp<DPP_MIRROR>(m), dpp<DPP_MIRROR>(am));
  if (GS > 16) take_larger(m, am, __shfl_xor(m, 16), __shfl_xor(am, 16));
  if (GS > 32) take_larger(m, am, __shfl_xor(m, 32), __shfl_xor(am, 32));
}

// Softmax cross-entropy of a batch, a group of GS >= R lanes per message and a class per lane: logits = the sum of the
// two halves za, zb; d logits to za, zero in an evaluation node.  (A thread per message, class after class, is 3000 cycles
// of dependent exponentials however few messages there are.)  A NaN logit makes the loss NaN; it is the prediction
// only as class 0's, which a comparison with it never replaces.
template <int GS>
__device__ __forceinline__ void softmax_batch(LDSQ float* za, const LDSQ float* zb, int ldz, int n, int R, const BatchMsg& M, GQ float* loss_out,
                                              GQ int* correct_out) {
  constexpr float INF = __builtin_inff();
  const int r = threadIdx.x & (GS - 1);
  for (int k = threadIdx.x / GS; k < n; k += AMP_THREADS / GS) {   // whole groups stay or leave
    const int label = M.a[k];
    const bool in = r < R;
    const float v = in ? za[k * ldz + r] + zb[k * ldz + r] : -INF;
    float m = v != v ? (r == 0 ? INF : -INF) : v;
    int am = in ? r : GS;
    group_argmax<GS>(m, am);
    const float e = in ? expf(v - m) : 0.f;
    const float se = group_sum<GS>(e);
    if (in) za[k * ldz + r] = M.aux[k] ? 0.f : e * (1.f / se) - (r == label ? 1.f : 0.f);
    if (r == label) {
      const unsigned idx = M.seq[k] - s_first_seq;
      __hip_atomic_fetch_add(loss_out + idx, -(v - m - logf(se)), __ATOMIC_RELAXED, AGENT);
      if (am == label) __hip_atomic_fetch_add(correct_out + idx, 1, __ATOMIC_RELAXED, AGENT);
    }
  }
}

template <int NG>
__device__ __noinline__ void role_tree_out(const GQ AmpDev* D, const GQ WorkerDev* W) {
  const GQ NodeDev& nd = D->node[3];
  const Tile t = make_tile(nd, W);
  const TreeBufs B = tree_bufs(D);
  const WorkerRegs wr = worker_regs(D, W);
  const int R = t.R, C = t.C, H = B.H, Hp = B.Hp, KB = wr.kb, ldw = t.ldw, nd_muf = uni(nd.muf);
  const int ldh = amp_ldrow(Hp), ldz = amp_ldrow(t.Rp), NRB = t.Rp >> 4, NCG = amp_round16(t.Cl) >> 4, SG = Hp >> 2;
  const GQ int* smeta = uni_gq<int>(D->smeta);
  const GQ int* tnode = uni_gq<int>(D->data.tnode);
  const GQ int* slot_inst = uni_gq<int>(D->slot_inst);
  GQ float* loss_out = uni_gq<float>(D->loss_out);
  GQ int* correct_out = uni_gq<int>(D->correct_out);
  GQ float* probe = uni_gq<float>(D->probe);
  GQ unsigned* probe_n = uni_gq<unsigned>(D->probe_n);
  const unsigned probe_period = uni(D->probe_period), probe_cap = uni(D->probe_cap);
  const int probe_w = uni(D->probe_w);
  const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  const SmallDiv by_ncg(NCG);
  typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));   // gout's rows are H floats apart
  Lds L{amp_lds};
  float* Wg = L.take(t.Rp * t.ldw);
  float* bg = L.take(t.Rp);
  LDSQ float* Wl = (LDSQ float*)Wg;
  LDSQ float* bl = (LDSQ float*)bg;
  LDSQ float* hbuf = (LDSQ float*)L.take(KB * ldh);   // per message: the node's h; the columns beyond it stay zero
  LDSQ float* zbuf = (LDSQ float*)L.take(KB * ldz);   // per message: logits over the first half of the columns, then d logits
  LDSQ float* zbuf2 = (LDSQ float*)L.take(KB * ldz);  // ... over the second half
  LDSQ int* done_cnt = (LDSQ int*)L.take(D->mak);     // eval: nodes scored per slot
  tile_load(nd, t, Wg, bg);
  for (int k = threadIdx.x; k < KB * ldh; k += AMP_THREADS) hbuf[k] = 0.f;
  for (int k = threadIdx.x; k < KB * ldz; k += AMP_THREADS) zbuf[k] = zbuf2[k] = 0.f;
  for (int k = threadIdx.x; k < D->mak; k += AMP_THREADS) done_cnt[k] = 0;
  // this thread's groups threadIdx.x - 128 + 384 j of the gradient -- four columns of a row, by waves 2..7 --, their optimizer
  // slots, and those of the bias of row threadIdx.x - 128
  constexpr int GT = AMP_THREADS - 128;
  const int gt = (int)threadIdx.x - 128, CG = (C + 3) >> 2;
  GQ float* ndG = uni_gq<float>(nd.G);
  GQ float* ndM = uni_gq<float>(nd.M);
  GQ float* ndV = uni_gq<float>(nd.V);
  const OptCoef ob = opt_base(nd);
  const bool mean = uni(nd.mean) != 0, bounded = uni(D->admit_bounded) != 0;
  unsigned count = W->wstate[0], tstep = W->wstate[1];
  v4f gacc[NG], sm[NG], sv[NG];
  float gb = 0.f, bm = 0.f, bv = 0.f;
  int er[NG], ec[NG];   // row (-1: no group) and first column
#pragma unroll
  for (int j = 0; j < NG; ++j) {
    const int e = gt + GT * j;
    const bool in = gt >= 0 && e < R * CG;
    er[j] = in ? e / CG : -1;
    ec[j] = in ? (e - (e / CG) * CG) << 2 : 0;
    gacc[j] = sm[j] = sv[j] = zero;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (in && ec[j] + v < C) {
        const int p = er[j] * C + ec[j] + v;
        gacc[j][v] = ndG[p];
        if (ob.kind != 0) sm[j][v] = ndM[p];
        if (ob.kind == 2) sv[j][v] = ndV[p];
      }
  }
  const bool bias = gt >= 0 && gt < R;
  if (bias) {
    gb = ndG[R * C + gt];
    if (ob.kind != 0) bm = ndM[R * C + gt];
    if (ob.kind == 2) bv = ndV[R * C + gt];
  }
  // Adam's powers b^t carried along in double precision
  double pw1 = ob.kind == 2 ? ipow((double)ob.b1, tstep) : 0.0, pw2 = ob.kind == 2 ? ipow((double)ob.b2, tstep) : 0.0;
  BatchMsg& M = s_M;
  __syncthreads();
  const Ring mine = ring_regs(D, uni(W->ring));
  unsigned head = 0;
  auto take_batch = [&](int room) {
    const int n = poll_batch(D, mine, head, KB, room, s_codes, &s_n, [](unsigned) { return true; });
    if (n > 0) {
      const int k = lane;
      if (k < n) {
        const unsigned code = s_codes[k];
        const int s = MSG_SLOT(code), nn = MSG_LOCAL(code);
        const v4i sl = tree_slot(smeta, s);
        const int word = slot_inst[s];
        const v4i tn = tree_node(tnode, sl.z, nn);
        M.s[k] = s;
        M.n[k] = nn;
        M.seq[k] = (unsigned)sl.x;
        M.a[k] = tn.w;
        M.par[k] = tn.z;
        M.L[k] = sl.y;
        // 1 = a node of an evaluation instance: scored, then counted towards the instance's retirement; no gradient
        M.aux[k] = (!wr.train || word < 0) ? 1 : 0;
        M.off0[k] = (int)(B.node(s, nn) * 2 * Hp);
        M.dst0[k] = (int)(B.node(s, nn) * H);
        // probe: this node's h (its cell's forward output) if the instance is sampled
        int entry = -1;
        if (probe_period && (unsigned)sl.x % probe_period == 0u) {
          const unsigned e = __hip_atomic_fetch_add(probe_n, 1u, __ATOMIC_RELAXED, AGENT);
          if (e < probe_cap) {
            entry = (int)e;
            GQ int* hdr = (GQ int*)(probe + (long long)e * probe_w);
            hdr[0] = 0;
            hdr[1] = sl.x;
            hdr[2] = nn;
            hdr[3] = 0;
          }
        }
        M.b[k] = entry;
      }
      // the event record: a training node's message is a forward event followed by a backward event (the loss turns
      // it round in place), an evaluation node's a forward event only
      const bool in = k < n, tr = in && M.aux[k] == 0;
      const unsigned long long mt = __ballot(tr);
      if (k == 0) M.nB = __popcll(mt);   // gradients in this batch
      if (wr.log_cap) {
        const unsigned base = s_logn, at = base + (unsigned)k + (unsigned)__popcll(mt & ((1ull << k) - 1ull));
        const unsigned total = (unsigned)n + (unsigned)__popcll(mt);
        if (base + total > wr.log_cap) {
          if (k == 0) raise_abort(D, ABORT_LOG_FULL, blockIdx.x);
        } else {
          if (in) {
            const unsigned long long tail = ((unsigned long long)M.seq[k] << 32) | (3ull << 20) | ((unsigned)M.n[k] & 0xfffffu);
            wr.log[at] = tail;
            if (tr) wr.log[at + 1] = tail | (1ull << 28);
          }
          if (k == 0) s_logn = base + total;
        }
      }
    }
  };
  if (wave == 1) take_batch(wr.train ? nd_muf - (int)count : KB_MAX);
  lds_barrier();
  for (;;) {
    const int n = uni(s_n);
    if (n == 0) break;
    head += n;
    const int NB = (n + 15) >> 4;
    // ---------------- h rows to LDS
    {
      const int ro = M.off0[lane];
      for (int r = wave; r < n; r += 8) {
        const GQ float* from = B.hc + __builtin_amdgcn_readlane(ro, r);
        for (int k = 0; k < SG; k += 64)
          if (k + lane < SG) global_to_lds(from + 4 * k, hbuf + r * ldh + 4 * k);
      }
      wait_vm();
    }
    lds_barrier();
    PHASE(0);
    if (probe_period)
      for (int idx = threadIdx.x; idx < n * SG; idx += AMP_THREADS) {
        const int k = idx / SG, c = (idx - k * SG) << 2;
        if (M.b[k] >= 0) *(GQ v4f*)(probe + (long long)M.b[k] * probe_w + 4 + c) = *(const LDSQ v4f*)(hbuf + k * ldh + c);
      }
    // ---------------- logits: item = (half of the columns, 16 classes, 16 messages)
    for (int it = wave; it < 2 * NRB * NB; it += AMP_THREADS / 64) {
      const int half = it & 1, rest = it >> 1, nb = rest / NRB, rb = rest - nb * NRB, j = nb * 16 + i, c0 = half ? NCG >> 1 : 0;
      const int nc = half ? NCG - (NCG >> 1) : NCG >> 1;
      v4f acc[4] = {half ? zero : *(const LDSQ v4f*)(bl + rb * 16 + 4 * q), zero, zero, zero};
      cell_rows(Wl + (rb * 16 + i) * ldw + 4 * q + 16 * c0, hbuf + (j < n ? j : n - 1) * ldh + 4 * q + 16 * c0, nc, acc);
      if (j < n) *(LDSQ v4f*)((half ? zbuf2 : zbuf) + j * ldz + rb * 16 + 4 * q) = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    }
    lds_barrier();
    PHASE(1);
    // ---------------- softmax cross-entropy; z becomes dz = p - onehot(label), zero in an evaluation node
    if (R <= 8)
      softmax_batch<8>(zbuf, zbuf2, ldz, n, R, M, loss_out, correct_out);
    else if (R <= 16)
      softmax_batch<16>(zbuf, zbuf2, ldz, n, R, M, loss_out, correct_out);
    else
      softmax_batch<64>(zbuf, zbuf2, ldz, n, R, M, loss_out, correct_out);
    PHASE(2);
    if (wr.train) {
      lds_barrier();
      // ---------------- dh[k][c] = sum_r W[r][c] dz[k][r]: item = (16 messages, 16 columns), four classes a step
      const int steps = (R + 3) >> 2;
      int nb_of = -1, j = 0;
      const LDSQ float* zp = zbuf;
      GQ float* to = B.gout;
      for (int it = wave; it < NB * NCG; it += AMP_THREADS / 64) {
        const int nb = by_ncg(it), cb = it - nb * NCG;
        if (nb != nb_of) {   // this lane's message
          nb_of = nb;
          j = nb * 16 + i;
          const int jj = j < n ? j : n - 1;
          zp = zbuf + jj * ldz + q;
          to = B.gout + M.dst0[jj] + 4 * q;
        }
        const LDSQ float* wp = Wl + q * ldw + cb * 16 + i;
        v4f a0 = zero, a1 = zero;
        for (int k = 0; k < steps; k += 2) {
          a0 = MFMA(wp[4 * k * ldw], zp[4 * k], a0);
          if (k + 1 < steps) a1 = MFMA(wp[4 * (k + 1) * ldw], zp[4 * (k + 1)], a1);
        }
        a0 += a1;
        const int c = cb * 16 + 4 * q;
        if (j < n) {
          if (c + 3 < C) {
            *(GQ v4fu*)(to + cb * 16) = a0;
          } else {
#pragma unroll
            for (int v = 0; v < 3; ++v)
              if (c + v < C) to[cb * 16 + v] = a0[v];
          }
        }
      }
    }
    PHASE(3);
    // what lane k of wave 0 needs of message k for its joins, before the batch's record is given up
    const int nB = uni(M.nB), jk = lane < n ? lane : 0;
    const int js = M.s[jk], jn = M.n[jk], jaux = M.aux[jk], jpar = M.par[jk], jL = M.L[jk];
    // every wave's HBM stores have landed before wave 0 publishes the batch
    publish_barrier();
    PHASE(4);
    const bool due = wr.train && (int)count + nB >= nd_muf;
    if (wave == 0) {
      fence_release();
      bool fin = false;
      if (lane < n && jaux) {
        fin = atomicAdd((int*)&done_cnt[js], 1) + 1 == 2 * jL - 1;
        if (fin) done_cnt[js] = 0;
      }
      tree_out_publish(wr, B, js, jn, lane < n && !jaux, jpar < 0, jn < jL, fin);
    }
    PHASE(5);
    if (wave == 1) {
      // recorded by the wave that records the next batch's events, so that the update comes first
      if (due && lane == 0) log_event(D, W, &s_logn, 3, 2, 0, 0);
      take_batch(wr.train ? nd_muf - (due ? 0 : (int)count + nB) : KB_MAX);
    }
    if (wr.train) {
      // ---------------- G[r][c] += sum_k dz[k][r] h[k][c], messages in ring order
#pragma unroll
      for (int j = 0; j < NG; ++j)
        if (er[j] >= 0) {
          const LDSQ float *zp = zbuf + er[j], *hp = hbuf + ec[j];
          int k = 0;
          for (; k + 3 < n; k += 4) {   // four messages' operands are read together, then added in ring order
            float zz[4];
            v4f hh[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              zz[b] = zp[(k + b) * ldz];
              hh[b] = *(const LDSQ v4f*)(hp + (k + b) * ldh);
            }
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
              for (int v = 0; v < 4; ++v) gacc[j][v] = fmaf(zz[b], hh[b][v], gacc[j][v]);
          }
          for (; k < n; ++k) {
            const float zz = zp[k * ldz];
            const v4f hh = *(const LDSQ v4f*)(hp + k * ldh);
#pragma unroll
            for (int v = 0; v < 4; ++v) gacc[j][v] = fmaf(zz, hh[v], gacc[j][v]);
          }
        }
      if (bias)
        for (int k = 0; k < n; ++k) gb += zbuf[k * ldz + gt];
      count += nB;
      if (due) {
        // ---------------- the node's own update (Section 3); every thread owns its elements, and the old weights have been read
        tstep++;
        if (bounded && threadIdx.x == 0) note_update(D);
        OptCoef o = ob;
        if (ob.kind == 2) {
          pw1 *= (double)ob.b1;
          pw2 *= (double)ob.b2;
          o.c1 = (float)(1.0 / (1.0 - pw1));
          o.c2 = (float)(1.0 / (1.0 - pw2));
        }
        const float inv = mean ? 1.f / (float)count : 1.f;
#pragma unroll
        for (int j = 0; j < NG; ++j)
          if (er[j] >= 0) {
            LDSQ v4f* wp = (LDSQ v4f*)(Wl + er[j] * ldw + ec[j]);
            v4f w = *wp;
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (ec[j] + v < C) {   // the columns beyond the row stay zero
                float m = sm[j][v], s = sv[j][v];
                w[v] = opt_step(o, w[v], gacc[j][v] * inv, m, s);
                sm[j][v] = m;
                sv[j][v] = s;
              }
            *wp = w;
            gacc[j] = zero;
          }
        if (bias) {
          bl[gt] = opt_step(o, bl[gt], gb * inv, bm, bv);
          gb = 0.f;
        }
        count = 0;
      }
    }
    PHASE(6);
    lds_barrier();
    PHASE(7);
  }
  tile_store(nd, t, Wg, bg);
#pragma unroll
  for (int j = 0; j < NG; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (er[j] >= 0 && ec[j] + v < C) {
        const int p = er[j] * C + ec[j] + v;
        ndG[p] = gacc[j][v];
        if (ob.kind != 0) ndM[p] = sm[j][v];
        if (ob.kind == 2) ndV[p] = sv[j][v];
      }
  if (bias) {
    ndG[R * C + gt] = gb;
    if (ob.kind != 0) ndM[R * C + gt] = bm;
    if (ob.kind == 2) ndV[R * C + gt] = bv;
  }
  if (threadIdx.x == 0) {
    W->wstate[0] = count;
    W->wstate[1] = tstep;
  }
}
