// Workers of the MLP: one per linear layer.
#pragma once

// Worker for linear layer `aux` (0..2) with its ReLU fused; the last layer
// also hosts the softmax loss, which turns the forward message round.
// Slot storage: buf[0]=act1, buf[1]=act2 (post-ReLU outputs), buf[2]=grad
// w.r.t. act1, buf[3]=grad w.r.t. act2.  Weights, bias and the gradient
// accumulator (same layout) stay in LDS for the life of the launch; the
// accumulator rests in HBM between launches.
__device__ __noinline__ void role_mlp_lin(const GQ AmpDev* D, const GQ WorkerDev* W) {
  float* lds = amp_lds;
  const GQ NodeDev& nd = D->node[uni(W->node)];
  const Tile t = make_tile(nd, W);
  const int R = t.R, C = t.C, li = uni(W->aux), ldw = t.ldw, muf = uni(nd.muf), train = uni(D->train);
  const bool first = li == 0, last = li == 2;
  Lds L{lds};
  float* Wg = L.take(t.Rp * ldw);
  float* bg = L.take(t.Rp);
  LDSQ float* Wl = (LDSQ float*)Wg;
  LDSQ float* bl = (LDSQ float*)bg;
  LDSQ float* Gl = (LDSQ float*)L.take(t.Rp * ldw);
  LDSQ float* gbl = (LDSQ float*)L.take(t.Rp);
  LDSQ float* xs = (LDSQ float*)L.take(ldw);
  LDSQ float* ys = (LDSQ float*)L.take(R);
  LDSQ float* ds = (LDSQ float*)L.take(R);
  LDSQ float* dx = (LDSQ float*)L.take(C);
  LDSQ float* part = (LDSQ float*)L.take(8 * (R > C ? R : C));
  tile_load(nd, t, Wg, bg);
  GQ float* ndG = uni_gq<float>(nd.G);
  GQ float* ndM = uni_gq<float>(nd.M);
  GQ float* ndV = uni_gq<float>(nd.V);
  const long long boff = (long long)uni(nd.rows) * C;
  const int has_bias = uni(nd.has_bias);
  for (int i = threadIdx.x; i < t.Rp * ldw; i += AMP_THREADS) {
    const int lr = i / ldw, c = i - lr * ldw;
    Gl[i] = (lr < R && c < C) ? ndG[(long long)lr * C + c] : 0.f;
  }
  for (int i = threadIdx.x; i < t.Rp; i += AMP_THREADS) gbl[i] = (i < R && has_bias) ? ndG[boff + i] : 0.f;
  for (int i = threadIdx.x; i < ldw; i += AMP_THREADS) xs[i] = 0.f;
  __syncthreads();
  const GQ float* act_in = first ? nullptr : uni_gq<float>(D->buf[li - 1]);
  GQ float* act_out = last ? nullptr : uni_gq<float>(D->buf[li]);
  const GQ float* g_in = last ? nullptr : uni_gq<float>(D->buf[2 + li]);
  GQ float* g_out = first ? nullptr : uni_gq<float>(D->buf[2 + li - 1]);
  const GQ float* datax = uni_gq<float>(D->data.x);
  const GQ int* lab = uni_gq<int>(D->data.lab);
  const GQ int* lab_off = uni_gq<int>(D->data.lab_off);
  const GQ unsigned* slot_seq = uni_gq<unsigned>(D->slot_seq);
  const GQ int* slot_inst = uni_gq<int>(D->slot_inst);
  GQ float* loss_out = uni_gq<float>(D->loss_out);
  GQ int* correct_out = uni_gq<int>(D->correct_out);
  const unsigned first_seq = uni(s_first_seq);
  const int ring = uni(W->ring);
  const Ring mine = ring_regs(D, ring), next = ring_regs(D, last ? ring : ring + 1), prev = ring_regs(D, ring - 1), ctl = ring_regs(D, 0);
  unsigned head = 0, code;
  unsigned count = W->wstate[0], tstep = W->wstate[1];
  while (wait_msg(D, mine, head, s_ctl, code)) {
    const int s = MSG_SLOT(code);
    const unsigned seq = uni(slot_seq[s]);
    const int word = uni(slot_inst[s]), inst = word & 0x7fffffff;
    const bool fwd_only = !train || word < 0;   // an evaluation instance: the loss layer retires it
    const GQ float* x = first ? datax + (long long)inst * C : act_in + (long long)s * C;
    bool backward = (code & MSG_DIR_B) != 0;
    for (int c = threadIdx.x; c < C; c += AMP_THREADS) xs[c] = x[c];
    if (backward)
      for (int r = threadIdx.x; r < R; r += AMP_THREADS)
        ds[r] = act_out[(long long)s * R + r] > 0.f ? g_in[(long long)s * R + r] : 0.f;
    lds_barrier();
    if (!backward) {
      gemv_rows(Wl, ldw, R, C, bl, xs, part, ys);
      LOG(W->node, 0, seq, 0);
      if (!last) {
        for (int r = threadIdx.x; r < R; r += AMP_THREADS) act_out[(long long)s * R + r] = fmaxf(ys[r], 0.f);
        publish_barrier();
        if (threadIdx.x == 0) {
          fence_release();
          ring_post(next, MSG_MAKE(0, s, 0));
        }
        continue;
      }
      const int label = lab[lab_off[inst]];
      softmax_xent_wave0((float*)ys, R, label, (float*)ds, &s_loss, &s_pred);
      if (threadIdx.x == 0) {
        loss_out[seq - first_seq] = s_loss;
        correct_out[seq - first_seq] = s_pred == label;
      }
      if (fwd_only) {
        publish_barrier();
        if (threadIdx.x == 0) {
          fence_release();
          ring_post(ctl, MSG_MAKE(1, s, 0));
        }
        continue;
      }
      backward = true;   // the loss layer starts backpropagation
    }
    LOG(W->node, 1, seq, 0);
    if (!first) {
      gemv_cols(Wl, ldw, R, C, ds, part, dx);
      for (int c = threadIdx.x; c < C; c += AMP_THREADS) g_out[(long long)s * C + c] = dx[c];
    }
    // every wave's HBM stores have landed before thread 0 publishes
    publish_barrier();
    if (threadIdx.x == 0) {
      fence_release();
      ring_post(prev, MSG_MAKE(1, s, 0));
    }
    tile_accumulate_lds(t, Gl, gbl, ds, xs);
    count++;
    if ((int)count >= muf) {
      // the node's own update (Section 3) from the accumulator in LDS
      tstep++;
      if (threadIdx.x == 0) note_update(D);
      lds_barrier();
      const OptCoef o = opt_coef(nd, tstep);
      const float inv = nd.mean ? 1.f / (float)count : 1.f;
      for (int i = threadIdx.x; i < R * ldw; i += AMP_THREADS) {
        const int lr = i / ldw, c = i - lr * ldw;
        if (c < C) {
          Wl[i] = opt_apply(o, Wl[i], Gl[i] * inv, ndM, ndV, (long long)lr * C + c);
          Gl[i] = 0.f;
        }
      }
      if (has_bias)
        for (int lr = threadIdx.x; lr < R; lr += AMP_THREADS) {
          bl[lr] = opt_apply(o, bl[lr], gbl[lr] * inv, ndM, ndV, boff + lr);
          gbl[lr] = 0.f;
        }
      count = 0;
      LOG(W->node, 2, 0, 0);
    }
    lds_barrier();
  }
  tile_store(nd, t, Wg, bg);
  for (int i = threadIdx.x; i < R * ldw; i += AMP_THREADS) {
    const int lr = i / ldw, c = i - lr * ldw;
    if (c < C) ndG[(long long)lr * C + c] = Gl[i];
  }
  if (has_bias)
    for (int lr = threadIdx.x; lr < R; lr += AMP_THREADS) ndG[boff + lr] = gbl[lr];
  if (threadIdx.x == 0) {
    W->wstate[0] = count;
    W->wstate[1] = tstep;
  }
}
