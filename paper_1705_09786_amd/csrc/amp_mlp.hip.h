// Workers of the MLP: one per linear layer `aux` (0..2) with its ReLU fused; the last layer also hosts the softmax
// loss, which turns the forward message round.  For the models that are not the work of one workgroup (mlp_one_fits in
// amp_mlp_one.hip.h has the rule and both sides' figures): inputs wider than 128, training with slots, and training with
// gradients to keep at more than 64 hidden units where the inputs are wider than 64 too or an update comes every two or three.
//
// Slot storage, rows of hidden rounded up to 4 floats: buf[0] = act1, buf[1] = act2 (post-ReLU outputs), buf[2] =
// gradient w.r.t. act1, buf[3] = gradient w.r.t. act2.
//
// Rings: 0 the controller's, 1 + l layer l's forward messages, 4 and 5 the backward messages of layers 0 and 1.  A
// worker looks at both of its rings at once and takes a waiting backward message first (Appendix A's priority).  Every
// ring but the controller's has a single producer, which keeps the tail in a register: a post is one store, where a
// shared tail costs an atomic's round trip (255 ns) in front of it.
#pragma once

struct MlpRings {
  Ring fwd, bwd, next, prev, ctl;
  unsigned fwd_head, bwd_head, next_tail, prev_tail, buf;
  unsigned long long waited;   // ticks
  unsigned messages;
};

__device__ __forceinline__ MlpRings mlp_rings(const GQ AmpDev* D, int li) {
  MlpRings q;
  q.fwd = ring_regs(D, 1 + li);
  q.bwd = ring_regs(D, li < 2 ? 4 + li : 1 + li);
  q.next = ring_regs(D, li < 2 ? 2 + li : 1 + li);
  q.prev = ring_regs(D, li > 0 ? 3 + li : 0);
  q.ctl = ring_regs(D, 0);
  q.fwd_head = q.bwd_head = q.next_tail = q.prev_tail = q.buf = q.messages = 0;
  q.waited = 0;
  return q;
}

// ONE thread, the ring's only producer.  near: every reader polls through this workgroup's L2.
__device__ __forceinline__ void mlp_post(bool near, const Ring& r, unsigned& tail, unsigned code) {
  if (near)
    ring_put_near(r, tail++, code);
  else
    ring_put(r, tail++, code);
}

__shared__ unsigned s_mlp[2][2];

// Whole workgroup: wave 0 polls both rings, everybody gets the code of the message taken; false when the run is over.
// Nothing is invalidated (but in the strict build): where s_nowb holds, the caller reads what it was sent with ld_shared.
__device__ __forceinline__ bool mlp_wait(const GQ AmpDev* D, MlpRings& q, unsigned& code) {
  unsigned* out = s_mlp[q.buf];   // two buffers: a wave may still read the one while wave 0 fills the other
  q.buf ^= 1u;
  if (threadIdx.x < 64) {
    const bool second = (threadIdx.x & 1) != 0;   // even lanes: backward ring, odd lanes: forward ring
    const unsigned head = second ? q.fwd_head : q.bwd_head;
    GQ unsigned long long* slot = second ? &q.fwd.ent[head & q.fwd.mask] : &q.bwd.ent[head & q.bwd.mask];
    const bool has_bwd = q.bwd.ent != q.fwd.ent;
    const long long t0 = wall_clock64();
    unsigned spins = 0, stop = 0;
    unsigned long long e, ready;
    for (;;) {
      e = __hip_atomic_load(slot, __ATOMIC_RELAXED, AGENT);
      ready = __ballot((unsigned)(e >> 32) == head + 1u && (second || has_bwd)) & 3ull;
      if (ready) break;
      if ((++spins & 15u) == 0u) {
        if (uni(ld_u32(&D->ctl[0]) | ld_u32(&D->ctl[1]))) {
          // done is only raised once nothing is in flight; look once more
          e = __hip_atomic_load(slot, __ATOMIC_RELAXED, AGENT);
          ready = __ballot((unsigned)(e >> 32) == head + 1u && (second || has_bwd)) & 3ull;
          if (ready && uni(ld_u32(&D->ctl[0])) == 0u) break;
          stop = 1;
          break;
        }
        if (uni((int)(wall_clock64() - t0 > D->watchdog_ticks))) {
          if (threadIdx.x == 0) raise_abort(D, ABORT_WATCHDOG, blockIdx.x);
          stop = 1;
          break;
        }
      }
    }
    const int lane = (ready & 1ull) ? 0 : 1;
    const unsigned taken = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)e, lane);
    q.waited += (unsigned long long)(wall_clock64() - t0);
    q.messages += 1u - stop;
    strict_acquire();
    if (threadIdx.x == 0) {
      out[0] = taken;
      out[1] = stop ? 0u : 1u + (unsigned)lane;
    }
  }
  lds_barrier();
  code = uni(out[0]);
  const unsigned from = uni(out[1]);
  q.bwd_head += from == 1u;
  q.fwd_head += from == 2u;
  return from != 0u;
}

// ------------------------------------------------------------ layers of up to 128 x 128: weights in registers
// A message costs this worker one matrix-vector product, so what bounds it is the chain of waits around it and the
// number of instructions its waves go through (about 4 cycles each, whatever they do).  With weights, gradient and update
// in LDS a 128 x 128 layer took 8.9 us per message, of which 33 rounds over the tile each for the accumulation and the
// update, with an integer division per element, were the most.  Here thread (wave w, cg = lane / 8, rg = lane % 8) keeps
// the weights of rows 32 w + 4 rg .. + 3 and columns 16 cg .. + 15 and their gradient in registers.  Forward: 64
// multiply-adds, then the four rows' sums over the eight column groups in seven instructions (a lane swap adds two
// rows at once and leaves each half of the wave with one of them).  Backward: 64 multiply-adds, sums over the row groups
// by DPP, over the waves through LDS.  A plain SGD update touches registers only.  Momentum and Adam have their slots
// in LDS and are dealt out element by element, 32 rows at a time, over all threads: a layer much smaller than 128 x 128
// leaves most lanes of the register layout without a weight, and an Adam step is some seventy instructions.
#define MLP_MAX 128   // rows and columns
#define MLP_GS (MLP_MAX + 4)   // row stride of the 32 rows an optimizer with slots works on at a time

// a of the lower and b of the upper half of the wave, each summed over the two halves.
__device__ __forceinline__ float swap_add32(float a, float b) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The same for the even and the odd 16-lane rows.
__device__ __forceinline__ float swap_add16(float a, float b) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float lane_of(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp<DPP_ROR8>(v);
  v += dpp<DPP_ROR4>(v);
  v += dpp<DPP_ROR2>(v);
  v += dpp<DPP_ROR1>(v);
  return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp<DPP_ROR8>(v));
  v = fmaxf(v, dpp<DPP_ROR4>(v));
  v = fmaxf(v, dpp<DPP_ROR2>(v));
  v = fmaxf(v, dpp<DPP_ROR1>(v));
  return fmaxf(fmaxf(lane_of(v, 0), lane_of(v, 16)), fmaxf(lane_of(v, 32), lane_of(v, 48)));
}

// Sixteen consecutive floats from p + at on, zero from index `end` on; `vec`: at and end are multiples of 4 and p is
// 16-byte aligned.
__device__ __forceinline__ void load_row(float (&v)[16], const GQ float* p, int at, int end, bool vec) {
  if (vec) {
#pragma unroll
    for (int k = 0; k < 16; k += 4) {
      const bool in = at + k < end;
      const v4f x = *(const GQ v4f*)(p + (in ? at + k : 0));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[k + e] = in ? x[e] : 0.f;
    }
  } else {
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const float x = p[at + k < end ? at + k : 0];
      v[k] = at + k < end ? x : 0.f;
    }
  }
}

// EACH: an update per gradient (min_update_frequency 1) under plain SGD, where the gradient needs no registers.  ADAPT:
// an optimizer with slots.  The loop has one path through it and changes the weights in one place: where several paths
// met, the compiler moved all 128 registers at each of them (0.6 us per message).
template <bool FIRST, bool LAST, bool EACH, bool ADAPT>
__device__ __noinline__ void role_mlp_regs(const GQ AmpDev* D, const GQ WorkerDev* W) {
  static_assert(AMP_THREADS == 256, "four waves of 32 rows");
  const GQ NodeDev& nd = D->node[uni(W->node)];
  const int R = uni(nd.rows), C = uni(nd.cols), HS = amp_round4(uni(D->hidden)), li = uni(W->aux), node = uni(W->node);
  const int muf = uni(nd.muf), train = uni(D->train), mean = uni(nd.mean);
  const float lr = uni(nd.lr);
  const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, rg = lane & 7, cg = lane >> 3;
  const int r0 = wave * 32 + 4 * rg, c0 = 16 * cg;
  const int my = r0 + (lane >> 5) + 2 * ((lane >> 4) & 1);   // the row whose sum this lane ends up with (twice per wave)
  const bool cvec = (C & 3) == 0;   // rows of C floats start 16-byte aligned
  const bool logging = uni(s_log_cap) != 0u;
  Lds L{amp_lds};
  LDSQ float* part = (LDSQ float*)L.take(4 * MLP_MAX);   // [wave][column] partial sums of W^T delta
  LDSQ float* zs = (LDSQ float*)L.take(64);              // logits
  LDSQ float* Ms = (LDSQ float*)L.take(MLP_MAX * MLP_MAX);   // optimizer slots [row][128]
  LDSQ float* Vs = (LDSQ float*)L.take(MLP_MAX * MLP_MAX);
  LDSQ float* Mb = (LDSQ float*)L.take(MLP_MAX);
  LDSQ float* Vb = (LDSQ float*)L.take(MLP_MAX);
  LDSQ float* gs = (LDSQ float*)L.take(32 * MLP_GS);   // gradients, then steps, of rows 4 x + a
  GQ float* P = uni_gq<float>(nd.P);
  GQ float* G = uni_gq<float>(nd.G);
  GQ float* M = uni_gq<float>(nd.M);
  GQ float* V = uni_gq<float>(nd.V);
  const int boff = R * C;
  float w[4][16], g[4][16], b, gb = 0.f;   // b, gb: bias of row `my` and its gradient
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const bool rin = r0 + a < R;
    const int row = rin ? (r0 + a) * C : 0, end = rin ? C : 0;
    load_row(w[a], P + row, c0, end, cvec);
    if (!EACH) load_row(g[a], G + row, c0, end, cvec);
  }
  b = my < R ? P[boff + my] : 0.f;
  if (!EACH) gb = my < R ? G[boff + my] : 0.f;
  const OptCoef ob = opt_base(nd);
  const int C4 = amp_round4(C);
  const bool whole = R * C4 <= 32 * MLP_GS;
  int csh = 0;   // columns rounded up to a power of two
  while ((1 << csh) < C) ++csh;
  if (ADAPT) {
    for (int e = threadIdx.x; e < R << csh; e += AMP_THREADS) {
      const int row = e >> csh, c = e & ((1 << csh) - 1);
      if (c < C) {
        Ms[row * MLP_MAX + c] = M[row * C + c];
        Vs[row * MLP_MAX + c] = V[row * C + c];
      }
    }
    Mb[my] = my < R ? M[boff + my] : 0.f;
    Vb[my] = my < R ? V[boff + my] : 0.f;
  }
  const GQ float* act_in = FIRST ? nullptr : uni_gq<float>(D->buf[li - 1]);
  GQ float* act_out = LAST ? nullptr : uni_gq<float>(D->buf[li]);
  const GQ float* g_in = LAST ? nullptr : uni_gq<float>(D->buf[2 + li]);
  GQ float* g_out = FIRST ? nullptr : uni_gq<float>(D->buf[2 + li - 1]);
  const GQ float* datax = uni_gq<float>(D->data.x);
  const GQ int* lab = uni_gq<int>(D->data.lab);
  const GQ unsigned* slot_seq = uni_gq<unsigned>(D->slot_seq);
  const GQ int* slot_inst = uni_gq<int>(D->slot_inst);
  GQ float* loss_out = uni_gq<float>(D->loss_out);
  GQ int* correct_out = uni_gq<int>(D->correct_out);
  const unsigned first_seq = uni(s_first_seq);
  // the storage rows' padding up to HS holds zeros; beyond it a row has nothing to read
  const int rin = r0 < HS ? r0 : 0;
  int cin[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) cin[k] = c0 + 4 * k < HS ? c0 + 4 * k : -1;
  MlpRings rq = mlp_rings(D, li);
  unsigned code, count = uni(W->wstate[0]), tstep = uni(W->wstate[1]);
  __syncthreads();
  while (mlp_wait(D, rq, code)) {
    const int s = MSG_SLOT(code), at = s * HS;
    const bool arrived_back = (code & MSG_DIR_B) != 0;
    const unsigned local = MSG_LOCAL(code);
    float x[16], d[4];
    int inst = (int)(local & MLP_LOOKUP);
    if ((FIRST || LAST) && inst == (int)MLP_LOOKUP) inst = uni(ld_shared(slot_inst + s)) & 0x7fffffff;
    // the layer's input; for a backward message also the gradient of its output and the output itself
    if (FIRST) {
      load_row(x, datax + (long long)inst * C, c0, C, cvec);
    } else {
      v4f t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = ld_shared4(act_in + at + (cin[k] < 0 ? 0 : cin[k]));
      // zero beyond the input, as load_row has it: the registers there are weights like any other to the updates below,
      // and a step with a zero input leaves them zero
#pragma unroll
      for (int k = 0; k < 16; ++k) x[k] = cin[k / 4] < 0 ? 0.f : t[k / 4][k & 3];
    }
    int label = 0;
    if (LAST) label = lab[inst];   // one label per instance
    unsigned seq = 0;
    if (LAST || logging) seq = ld_shared(slot_seq + s);
    // does this message go backward through the layer (the last layer turns training instances round)
    const bool back = LAST ? train && !(local & 0x80000u) : arrived_back;
    if (LAST || !arrived_back) {
      float y[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int k = 0; k < 16; k += 2) {
          s0 = fmaf(w[a][k], x[k], s0);
          s1 = fmaf(w[a][k + 1], x[k + 1], s1);
        }
        y[a] = s0 + s1;
      }
      float v = swap_add16(swap_add32(y[0], y[1]), swap_add32(y[2], y[3]));
      v += dpp<DPP_ROR8>(v);
      v += b;
      if (logging) LOG(node, 0, seq, 0);
      if (LAST) {
        // softmax cross-entropy: every wave for itself, lane k = class k
        if ((lane & 8) == 0 && my < 64) zs[my] = v;
        lds_barrier();
        const float z = lane < R ? zs[lane] : -3.0e38f;
        const float m = wave_max(z);
        const float e = lane < R ? expf(z - m) : 0.f;
        const float se = wave_sum(e);
        const float dz = lane < R ? e / se - (lane == label ? 1.f : 0.f) : 0.f;
        if (wave == 3) {   // not among the waves that write the result below
          const unsigned long long top = __ballot(lane < R && z == m);   // none where every logit is NaN
          const int best = top ? __builtin_ctzll(top) : 0;   // the first class with the largest logit
          const float zl = lane_of(z, uni(label));
          if (lane == 0) {
            loss_out[seq - first_seq] = -(zl - m - logf(se));
            correct_out[seq - first_seq] = best == label;
          }
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const float u = __int_as_float(__builtin_amdgcn_ds_bpermute(((r0 + a) & 63) << 2, __float_as_int(dz)));
          d[a] = r0 + a < R ? u : 0.f;
        }
      } else if ((lane & 8) == 0 && my < R) {
        act_out[at + my] = fmaxf(v, 0.f);
      }
    }
    if (back) {
      if (!LAST) {
        const v4f go = ld_shared4(g_in + at + rin), ao = *(const GQ v4f*)(act_out + at + rin);
#pragma unroll
        for (int a = 0; a < 4; ++a) d[a] = (r0 + a < R && ao[a] > 0.f) ? go[a] : 0.f;
      }
      if (logging) LOG(node, 1, seq, 0);
      if (!FIRST) {
        // W^T delta over this thread's rows, the wave's eight row groups, the waves that hold rows
        float p[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          p[k] = w[0][k] * d[0];
#pragma unroll
          for (int a = 1; a < 4; ++a) p[k] = fmaf(w[a][k], d[a], p[k]);
          p[k] += dpp<DPP_XOR1>(p[k]);
          p[k] += dpp<DPP_XOR2>(p[k]);
          p[k] += dpp<DPP_HALF_MIRROR>(p[k]);
        }
        if (rg == 0) {
#pragma unroll
          for (int k = 0; k < 16; k += 4) *(LDSQ v4f*)(part + wave * MLP_MAX + c0 + k) = (v4f){p[k], p[k + 1], p[k + 2], p[k + 3]};
        }
        lds_barrier();
        if ((int)threadIdx.x < C)
          g_out[at + threadIdx.x] = (part[threadIdx.x] + part[MLP_MAX + threadIdx.x]) +
                                    (part[2 * MLP_MAX + threadIdx.x] + part[3 * MLP_MAX + threadIdx.x]);
      }
    }
    // every wave has what it needs of the slot (the post may end the instance's life) and its stores have landed
    publish_barrier();
    if (threadIdx.x == 0) {
      if (back && !FIRST)
        mlp_post(true, rq.prev, rq.prev_tail, MSG_MAKE(1, s, local));
      else if (LAST || back) {
        strict_release();
        ring_post(rq.ctl, MSG_MAKE(1, s, 0));   // done: an evaluation instance, or back at the first layer
      } else
        mlp_post(true, rq.next, rq.next_tail, MSG_MAKE(0, s, local));
    }
    // the gradient; the node's own update (Section 3) when enough of them have arrived
    if (back) {
      const float dmy = (lane & 32) ? ((lane & 16) ? d[3] : d[1]) : ((lane & 16) ? d[2] : d[0]);   // delta of row `my`
      if (EACH) {
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const float step = -lr * d[a];
#pragma unroll
          for (int k = 0; k < 16; ++k) w[a][k] = fmaf(step, x[k], w[a][k]);
        }
        b = fmaf(-lr, dmy, b);
        tstep++;
        if (threadIdx.x == 0) note_update(D);
        if (logging) LOG(node, 2, 0, 0);
      } else {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int k = 0; k < 16; ++k) g[a][k] = fmaf(d[a], x[k], g[a][k]);
        gb += dmy;
        if ((int)++count >= muf) {
          tstep++;
          if (threadIdx.x == 0) note_update(D);
          const float inv = mean ? 1.f / (float)count : 1.f;
          if (!ADAPT) {
            const float step = -lr * inv;
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
              for (int k = 0; k < 16; ++k) {
                w[a][k] = fmaf(step, g[a][k], w[a][k]);
                g[a][k] = 0.f;
              }
            b = fmaf(step, gb, b);
          } else {
            const OptCoef o = opt_at(ob, tstep);
            // the layer at once where it fits, otherwise rows 4 x + a for a = 0 .. 3: row = row0 + rstep * (row in gs)
            auto step_rows = [&](int n_rows, int row0, int rstep, int gstride) {
              const int n = n_rows << csh, cmask = (1 << csh) - 1;
              for (int e0 = threadIdx.x; e0 < n; e0 += 4 * AMP_THREADS) {   // four elements in flight
                float gv[4], m1[4], v1[4];
                int gi[4], si[4];
                bool in[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                  const int e = e0 + u * AMP_THREADS, c = e & cmask;
                  in[u] = e < n && c < C;
                  gi[u] = in[u] ? (e >> csh) * gstride + c : 0;
                  si[u] = in[u] ? (row0 + rstep * (e >> csh)) * MLP_MAX + c : 0;
                  gv[u] = gs[gi[u]];
                  m1[u] = Ms[si[u]];
                  v1[u] = Vs[si[u]];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                  const float t = opt_step(o, 0.f, gv[u] * inv, m1[u], v1[u]);
                  if (in[u]) {
                    gs[gi[u]] = t;
                    Ms[si[u]] = m1[u];
                    Vs[si[u]] = v1[u];
                  }
                }
              }
            };
            if (whole) {
#pragma unroll
              for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int k = 0; k < 16; k += 4)
                  if (r0 + a < R && c0 + k < C4)
                    *(LDSQ v4f*)(gs + (r0 + a) * C4 + c0 + k) = (v4f){g[a][k], g[a][k + 1], g[a][k + 2], g[a][k + 3]};
              lds_barrier();
              step_rows(R, 0, 1, C4);
              lds_barrier();
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) {
              if (!whole) {
                lds_barrier();   // the previous rows' steps have been taken
#pragma unroll
                for (int k = 0; k < 16; k += 4)
                  *(LDSQ v4f*)(gs + (r0 >> 2) * MLP_GS + c0 + k) = (v4f){g[a][k], g[a][k + 1], g[a][k + 2], g[a][k + 3]};
                lds_barrier();
                step_rows((R - a + 3) >> 2, a, 4, MLP_GS);
                lds_barrier();
              }
              const LDSQ float* from = whole ? gs + (r0 + a < R ? r0 + a : 0) * C4 : gs + (r0 >> 2) * MLP_GS;
#pragma unroll
              for (int k = 0; k < 16; k += 4) {
                const v4f t = *(const LDSQ v4f*)(from + (c0 + k < C ? c0 + k : 0));
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  w[a][k + q] += (r0 + a < R && c0 + k + q < C) ? t[q] : 0.f;
                  g[a][k + q] = 0.f;
                }
              }
            }
            float m1 = Mb[my], v1 = Vb[my];
            b = opt_step(o, b, gb * inv, m1, v1);
            Mb[my] = m1;   // both lanes of the row hold the same values
            Vb[my] = v1;
          }
          gb = 0.f;
          count = 0;
          if (logging) LOG(node, 2, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    if (r0 + a >= R) continue;
    const int row = (r0 + a) * C;
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (c0 + k < C) {
        P[row + c0 + k] = w[a][k];
        if (!EACH) G[row + c0 + k] = g[a][k];
      }
  }
  if (ADAPT)
    for (int e = threadIdx.x; e < R << csh; e += AMP_THREADS) {
      const int row = e >> csh, c = e & ((1 << csh) - 1);
      if (c < C) {
        M[row * C + c] = Ms[row * MLP_MAX + c];
        V[row * C + c] = Vs[row * MLP_MAX + c];
      }
    }
  if ((lane & 8) == 0 && my < R) {
    P[boff + my] = b;
    if (!EACH) G[boff + my] = gb;
    if (ADAPT) {
      M[boff + my] = Mb[my];
      V[boff + my] = Vb[my];
    }
  }
  if (threadIdx.x == 0) {
    W->wstate[0] = count;
    W->wstate[1] = tstep;
    s_stat[0] = rq.waited;
    s_stat[1] = rq.messages;
  }
}

template <bool FIRST, bool LAST>
__device__ __forceinline__ void role_mlp_layer(const GQ AmpDev* D, const GQ WorkerDev* W) {
  const GQ NodeDev& nd = D->node[W->node];
  if (nd.opt != 0)
    role_mlp_regs<FIRST, LAST, false, true>(D, W);
  else if (nd.muf == 1 && W->wstate[0] == 0u)
    role_mlp_regs<FIRST, LAST, true, false>(D, W);
  else
    role_mlp_regs<FIRST, LAST, false, false>(D, W);
}

// ------------------------------------------------------------ a first layer of more than 128 inputs
// Weights, bias and the gradient accumulator (same layout) stay in LDS for the life of the launch; the accumulator rests
// in HBM between launches.  Only the first layer can be that large: a hidden layer beyond 128 x 128 does not fit the LDS
// twice, and the host refuses it.
//
// What bounds it: the passes over the tile, one per gradient and one per update.  Each thread takes four neighbouring
// elements at a time and steps row and column along with the index.  Element by element, with a division by the row
// length for each, an update per gradient took 21.1 us per instance at 64 x 200 with these 256 threads (15.3 with the 512
// of the other models' kernels); this takes 12.1, and at 16 x 784 12.6 instead of 21.1 (15.5 with 512).
__device__ __noinline__ void role_mlp_wide(const GQ AmpDev* D, const GQ WorkerDev* W) {
  float* lds = amp_lds;
  const GQ NodeDev& nd = D->node[uni(W->node)];
  const Tile t = make_tile(nd, W);
  const int HS = amp_round4(uni(D->hidden));   // row stride of the slot storage
  const int R = t.R, C = t.C, ldw = t.ldw, muf = uni(nd.muf);
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
  LDSQ float* part = (LDSQ float*)L.take(8 * R);
  tile_load(nd, t, Wg, bg);
  GQ float* ndG = uni_gq<float>(nd.G);
  GQ float* ndM = uni_gq<float>(nd.M);
  GQ float* ndV = uni_gq<float>(nd.V);
  const int boff = R * C;
  for (int i = threadIdx.x; i < t.Rp * ldw; i += AMP_THREADS) {
    const int lr = i / ldw, c = i - lr * ldw;
    Gl[i] = (lr < R && c < C) ? ndG[lr * C + c] : 0.f;
  }
  for (int i = threadIdx.x; i < t.Rp; i += AMP_THREADS) gbl[i] = i < R ? ndG[boff + i] : 0.f;
  for (int i = threadIdx.x; i < ldw; i += AMP_THREADS) xs[i] = 0.f;
  __syncthreads();
  GQ float* act_out = uni_gq<float>(D->buf[0]);
  const GQ float* g_in = uni_gq<float>(D->buf[2]);
  const GQ float* datax = uni_gq<float>(D->data.x);
  const GQ unsigned* slot_seq = uni_gq<unsigned>(D->slot_seq);
  const GQ int* slot_inst = uni_gq<int>(D->slot_inst);
  const OptCoef ob = opt_base(nd);
  const int mean = uni(nd.mean);
  // this thread's first group of four elements and the way from one to the next (rows of ldw / 4 groups)
  const int lq = ldw >> 2, row0 = (int)threadIdx.x / lq, cq0 = (int)threadIdx.x - row0 * lq;
  const int drow = AMP_THREADS / lq, dcq = AMP_THREADS - drow * lq;
#define MLP_FOR_GROUPS                                                                              \
  for (int q = threadIdx.x, lr = row0, cq = cq0; q < R * lq;                                        \
       q += AMP_THREADS, cq += dcq, lr += drow + (cq >= lq ? 1 : 0), cq -= cq >= lq ? lq : 0)
  MlpRings rq = mlp_rings(D, 0);
  unsigned code;
  unsigned count = W->wstate[0], tstep = W->wstate[1];
  while (mlp_wait(D, rq, code)) {
    // this path reads its inputs through the L1
    if (threadIdx.x == 0) fence_acquire();
    lds_barrier();
    const int s = MSG_SLOT(code);
    const unsigned seq = uni(slot_seq[s]);
    const int inst = uni(slot_inst[s]) & 0x7fffffff;
    const GQ float* x = datax + (long long)inst * C;
    const bool backward = (code & MSG_DIR_B) != 0;
    for (int c = threadIdx.x; c < C; c += AMP_THREADS) xs[c] = x[c];
    if (backward)
      for (int r = threadIdx.x; r < R; r += AMP_THREADS)
        ds[r] = act_out[(long long)s * HS + r] > 0.f ? g_in[(long long)s * HS + r] : 0.f;
    lds_barrier();
    if (!backward) {
      gemv_rows(Wl, ldw, R, C, bl, xs, part, ys);
      LOG(W->node, 0, seq, 0);
      for (int r = threadIdx.x; r < R; r += AMP_THREADS) act_out[(long long)s * HS + r] = fmaxf(ys[r], 0.f);
      publish_barrier();
      if (threadIdx.x == 0) {
        fence_release();
        mlp_post(false, rq.next, rq.next_tail, MSG_MAKE(0, s, MSG_LOCAL(code)));
      }
      continue;
    }
    LOG(W->node, 1, seq, 0);
    if (threadIdx.x == 0) {
      strict_release();
      ring_post(rq.ctl, MSG_MAKE(1, s, 0));   // retired: what it left is in LDS now
    }
    MLP_FOR_GROUPS {
      LDSQ v4f* g = (LDSQ v4f*)Gl + q;
      const v4f x4 = ((const LDSQ v4f*)xs)[cq];
      const float d = ds[lr];
      v4f a = *g;
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = fmaf(d, x4[e], a[e]);
      *g = a;
    }
    for (int lr = threadIdx.x; lr < R; lr += AMP_THREADS) gbl[lr] += ds[lr];
    count++;
    if ((int)count >= muf) {
      // the node's own update (Section 3) from the accumulator in LDS; every thread steps the elements it has summed
      tstep++;
      if (threadIdx.x == 0) note_update(D);
      const OptCoef o = opt_at(ob, tstep);
      const float inv = mean ? 1.f / (float)count : 1.f;
      MLP_FOR_GROUPS {
        LDSQ v4f *g = (LDSQ v4f*)Gl + q, *w = (LDSQ v4f*)Wl + q;
        v4f ga = *g, wa = *w;
        float m[4], v[4];
        const int at = lr * C + 4 * cq;
        if (o.kind != 0) {   // the slots are in HBM, all eight fetched together
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            m[e] = ndM[4 * cq + e < C ? at + e : 0];
            v[e] = o.kind == 2 ? ndV[4 * cq + e < C ? at + e : 0] : 0.f;
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float stepped = opt_step(o, wa[e], ga[e] * inv, m[e], v[e]);
          if (4 * cq + e < C) wa[e] = stepped;   // the padding stays zero, whatever slots it was stepped with
          if (o.kind != 0 && 4 * cq + e < C) {
            ndM[at + e] = m[e];
            if (o.kind == 2) ndV[at + e] = v[e];
          }
        }
        *w = wa;
        *g = (v4f){0.f, 0.f, 0.f, 0.f};
      }
      for (int lr = threadIdx.x; lr < R; lr += AMP_THREADS) {
        bl[lr] = opt_apply(o, bl[lr], gbl[lr] * inv, ndM, ndV, boff + lr);
        gbl[lr] = 0.f;
      }
      count = 0;
      LOG(W->node, 2, 0, 0);
    }
  }
#undef MLP_FOR_GROUPS
  tile_store(nd, t, Wg, bg);
  for (int i = threadIdx.x; i < R * ldw; i += AMP_THREADS) {
    const int lr = i / ldw, c = i - lr * ldw;
    if (c < C) ndG[lr * C + c] = Gl[i];
  }
  for (int lr = threadIdx.x; lr < R; lr += AMP_THREADS) ndG[boff + lr] = gbl[lr];
  if (threadIdx.x == 0) {
    W->wstate[0] = count;
    W->wstate[1] = tstep;
    s_stat[0] = rq.waited;
    s_stat[1] = rq.messages;
  }
}

__device__ __forceinline__ void role_mlp_lin(const GQ AmpDev* D, const GQ WorkerDev* W) {
  const GQ NodeDev& nd = D->node[W->node];
  if (!s_nowb) {   // four workers a replica are packed at every number of replicas; the hand-overs rely on it
    if (threadIdx.x == 0) raise_abort(D, ABORT_BAD_STATE, blockIdx.x);
  } else if (W->aux == 0 && nd.cols > MLP_MAX)
    role_mlp_wide(D, W);
  else if (W->aux == 0)
    role_mlp_layer<true, false>(D, W);
  else if (W->aux == 1)
    role_mlp_layer<false, false>(D, W);
  else
    role_mlp_layer<false, true>(D, W);
}
