// Leaf and branch cells whose tile keeps its weights in LDS (the streamed cells are role_tree_cell).
//
// A batch is a chain of short steps, each as long as its memory latency, its matrix time or its instructions:
//   gather   the inputs of all messages go from the slot storage straight to LDS rows, each line fetched once, while
//            the threads fetch and form the backward messages' deltas;
//   products the gradient's units, each by the wave that owns it, then forward (16 rows x 16 messages) and input-gradient
//            (16 columns x 32 messages) items from one list, taken by the waves as they get free: no kind of product alone
//            fills the four matrix pipes evenly;
//   outputs  activations of the forward messages;
//   publish  wave 0 joins and posts, wave 1 takes and decodes the next batch; the others make the update when the node's
//            count is reached.
// The accumulator -- the sum over messages of delta (x) input, the tile's share of the node's gradient -- stays in
// registers from one update to the next (16 floats a lane for a 16 x 64 unit), and with at most two units a wave the
// optimizer's slots do as well; between launches both rest in the node's arrays in HBM.
//
// On gfx950 a wave that issues fp32 matrix instructions back to back keeps every other wave of its SIMD from issuing
// vector instructions, whatever their priorities (measured: a wave of v_add beside one of 16x16x4 products stands still
// until those have finished).  So vector instructions cost matrix time and the other way round: addresses are scalar or
// computed once per batch, operands are selected by address and not by value, and no products are made beside the
// hand-over (the gradient's there stopped its two waves: 7 to 9 thousand cycles instead of 4).
#pragma once

__shared__ int s_item;   // next item of the running batch's products

// x / d for small x (x * d < 2^31): one multiplication.
struct SmallDiv {
  unsigned m;
  __device__ __forceinline__ explicit SmallDiv(int d) : m(d > 1 ? 0xffffffffu / (unsigned)d + 1u : 0u) {}
  __device__ __forceinline__ int operator()(int x) const { return m ? (int)__umulhi((unsigned)x, m) : x; }
};

// Four accumulators += W[r][c] x_j[c] over NCG 16-column groups, operands from LDS: the next four groups' operands are read while
// the present four go through the matrix core.
__device__ __forceinline__ void cell_rows(const LDSQ float* wp, const LDSQ float* xp, int NCG, v4f (&acc)[4]) {
  v4f w0[4], x0[4], w1[4], x1[4];
  auto fetch = [&](int c, v4f (&w)[4], v4f (&x)[4]) {   // four groups; the last four where fewer are left
    const int o = 16 * (c + 4 <= NCG ? c : NCG >= 4 ? NCG - 4 : 0);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      w[a] = *(const LDSQ v4f*)(wp + o + 16 * a);
      x[a] = *(const LDSQ v4f*)(xp + o + 16 * a);
    }
  };
  auto work = [&](v4f (&w)[4], v4f (&x)[4]) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = MFMA(w[a][e], x[a][e], acc[e]);
  };
  const int full = NCG >> 2;
  if (full > 0) fetch(0, w0, x0);
  for (int c = 0; c < full; c += 2) {
    fetch(4 * c + 4, w1, x1);
    asm volatile("" ::: "memory");
    work(w0, x0);
    if (c + 1 >= full) break;
    fetch(4 * c + 8, w0, x0);
    asm volatile("" ::: "memory");
    work(w1, x1);
  }
  for (int c = full << 2; c < NCG; ++c) {
    const v4f w = *(const LDSQ v4f*)(wp + 16 * c), x = *(const LDSQ v4f*)(xp + 16 * c);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = MFMA(w[e], x[e], acc[e]);
  }
}

// dx[b] = W^T delta for one 16-column group and NB blocks of messages (delta rows d0, d1).
template <int NB>
__device__ __forceinline__ void cell_cols(const LDSQ float* wp, int ldw, const LDSQ float* d0, const LDSQ float* d1, int NRB, v4f (&dx)[2]) {
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  struct Op {
    float w[4];
    v4f d[NB];
  };
  v4f acc[2][2] = {{zero, zero}, {zero, zero}};
  auto fetch = [&](int r, Op& o) {
    const int g = r < NRB ? r : NRB - 1;
#pragma unroll
    for (int e = 0; e < 4; ++e) o.w[e] = wp[(16 * g + e) * ldw];
    o.d[0] = *(const LDSQ v4f*)(d0 + 16 * g);
    if (NB == 2) o.d[NB - 1] = *(const LDSQ v4f*)(d1 + 16 * g);
  };
  auto work = [&](const Op& o) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[NB == 2 ? b : e >> 1][e & 1] = MFMA(o.w[e], o.d[b][e], acc[NB == 2 ? b : e >> 1][e & 1]);
  };
  Op o0, o1, o2;
  fetch(0, o0);
  fetch(1, o1);
  for (int r = 0; r < NRB; r += 3) {
    fetch(r + 2, o2);
    asm volatile("" ::: "memory");
    work(o0);
    if (r + 1 >= NRB) break;
    fetch(r + 3, o0);
    asm volatile("" ::: "memory");
    work(o1);
    if (r + 2 >= NRB) break;
    fetch(r + 4, o1);
    asm volatile("" ::: "memory");
    work(o2);
  }
  dx[0] = acc[0][0] + acc[0][1];
  dx[1] = acc[1][0] + acc[1][1];
  if (NB == 1) dx[0] += dx[1];
}

template <bool BR, int GU, int OPT>
__device__ __noinline__ void role_tree_cell_lds(const GQ AmpDev* D, const GQ WorkerDev* W) {
  const GQ NodeDev& nd = D->node[W->node];
  const Tile t = make_tile(nd, W);
  const TreeBufs B = tree_bufs(D);
  const WorkerRegs wr = worker_regs(D, W);
  const int R = t.R, H = B.H, Hp = B.Hp, nu = t.nu, u0 = t.u0, KB = wr.kb, nd_muf = uni(nd.muf);
  const GQ int* smeta = uni_gq<int>(D->smeta);
  const GQ int* tnode = uni_gq<int>(D->data.tnode);
  const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
  const int NRB = t.Rp >> 4, Cp = amp_round16(t.Cl), NCG = Cp >> 4, NU = NRB * ((Cp + 63) >> 6);
  const int ldw = t.ldw, ldy = amp_ldrow(R);
  const int SG = (BR ? t.segp : t.Cl) >> 2;   // 16-byte groups of an input segment
  const SmallDiv by_nu(nu), by_nrb(NRB);
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  Lds L{amp_lds};
  float* Wg = L.take(t.Rp * ldw);
  float* bg = L.take(t.Rp);
  LDSQ float* Wl = (LDSQ float*)Wg;
  LDSQ float* bl = (LDSQ float*)bg;
  // Row r of the batch: forward messages first, then the backward ones, each in ring order.
  LDSQ float* X = (LDSQ float*)L.take(KB * ldw);   // inputs, laid out like a row of the weights
  LDSQ float* Y = (LDSQ float*)L.take(KB * ldy);   // forward: pre-activations; backward: deltas
  LDSQ float* Z = (LDSQ float*)L.take(t.Rp);       // zeros
  LDSQ int* rowmap = (LDSQ int*)L.take(t.Rp);      // node row of a tile row, node column of an LDS column (-1 = padding)
  LDSQ int* colmap = (LDSQ int*)L.take(((Cp + 63) >> 6) << 6);
  tile_load(nd, t, Wg, bg);
  for (int k = threadIdx.x; k < KB * ldw; k += AMP_THREADS) X[k] = 0.f;   // the columns beyond the input stay zero
  for (int k = threadIdx.x; k < KB * ldy; k += AMP_THREADS) Y[k] = 0.f;
  for (int k = threadIdx.x; k < t.Rp; k += AMP_THREADS) Z[k] = 0.f;
  for (int k = threadIdx.x; k < t.Rp; k += AMP_THREADS) rowmap[k] = k < R ? t.grow(k) : -1;
  for (int k = threadIdx.x; k < ((Cp + 63) >> 6) << 6; k += AMP_THREADS) colmap[k] = t.ncol(k);
  __syncthreads();
  BatchMsg& M = s_M;
  const Ring mine = ring_regs(D, uni(W->ring));
  const GQ float* xbase = BR ? B.hc : B.xin;
  GQ float* obase = BR ? B.gpar : B.gx;
  unsigned head = 0, count = W->wstate[0], tstep = W->wstate[1];

  // ---- gradient accumulator.  Unit = (16-row block, 64-column block); unit u of a wave is wave * GU + u in column-block
  // order, so that the units of a wave share inputs
  auto unit_of = [&](int u) { return wave * GU + u < NU ? wave * GU + u : -1; };
  constexpr bool KEEP = GU <= 2;   // optimizer slots in registers
  const OptCoef ob = opt_base(nd);
  const bool slots = wr.train && OPT != 0;
  GQ float* ndG = uni_gq<float>(nd.G);
  GQ float* ndM = uni_gq<float>(nd.M);
  GQ float* ndV = uni_gq<float>(nd.V);
  v4f g[GU][4], sm[KEEP ? GU : 1][4], sv[KEEP && OPT == 2 ? GU : 1][4];   // [unit][column of the lane's four][row of its four]
  int arow[GU], xcol[GU];
  unsigned valid[GU];   // bit 4 v + e: a real element of the node
  auto at = [&](int u, int v, int e) {   // its place in the node's arrays
    const int id = unit_of(u), cm = by_nrb(id), rb = id - cm * NRB;
    return rowmap[rb * 16 + 4 * q + e] * t.C + colmap[cm * 64 + 4 * i + v];
  };
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const int id = unit_of(u) < 0 ? 0 : unit_of(u), cm = by_nrb(id), rb = id - cm * NRB, lc = cm * 64 + 4 * i;
    arow[u] = rb * 16;
    xcol[u] = lc < Cp ? lc : ldw - 4;   // beyond the row: its last four columns, always zero
    valid[u] = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      g[u][v] = zero;
      if (KEEP) sm[KEEP ? u : 0][v] = zero;
      if (KEEP && OPT == 2) sv[KEEP && OPT == 2 ? u : 0][v] = zero;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (unit_of(u) >= 0 && rowmap[rb * 16 + 4 * q + e] >= 0 && colmap[lc + v] >= 0) {
          valid[u] |= 1u << (4 * v + e);
          const int p = at(u, v, e);
          if (count > 0) g[u][v][e] = ndG[p];
          if (KEEP && slots) sm[KEEP ? u : 0][v][e] = ndM[p];
          if (KEEP && OPT == 2 && slots) sv[KEEP && OPT == 2 ? u : 0][v][e] = ndV[p];
        }
    }
  }
  // bias gradient and slots: rows threadIdx.x - 256 and threadIdx.x of the tile, by waves 4..7
  constexpr int BS = AMP_THREADS / 2;
  const int brow = (int)threadIdx.x - BS;
  float gb[2] = {0.f, 0.f}, bm[2] = {0.f, 0.f}, bv[2] = {0.f, 0.f};
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int r = brow + a * BS;
    if (brow >= 0 && r < R && nd.has_bias) {
      const int p = nd.rows * t.C + rowmap[r];
      if (count > 0) gb[a] = ndG[p];
      if (slots) bm[a] = ndM[p];
      if (slots && OPT == 2) bv[a] = ndV[p];
    }
  }
  // Adam's powers b^t carried along in double precision: a power per update instead of a product of its squares.  The next
  // update's factors are formed while a batch's inputs are on their way.
  double pw1 = OPT == 2 ? ipow((double)ob.b1, tstep) : 0.0, pw2 = OPT == 2 ? ipow((double)ob.b2, tstep) : 0.0;

  float c1 = 1.f, c2 = 1.f;
  bool formed = false;
  auto take_batch = [&](unsigned held) {
    if (lane == 0) s_item = 0;
    tree_take<BR>(D, wr, B, mine, head, nd_muf - (int)held, smeta, tnode);
  };
  if (wave == 1) take_batch(count);
  lds_barrier();
  for (;;) {
    const int n = uni(s_n);
    if (n == 0) break;
    head += n;
    const int nF = uni(M.nF), nB = n - nF;
    // ---------------- gather
    // inputs: rows of a wave at scalar addresses, up to 64 groups of 16 bytes of a segment per instruction, to LDS
    {
      const int ro0 = M.off0[lane], ro1 = M.off1[lane];
      for (int r = wave; r < n; r += 8) {
        const GQ float* s0 = xbase + __builtin_amdgcn_readlane(ro0, r);
        const GQ float* s1 = xbase + __builtin_amdgcn_readlane(ro1, r);
        LDSQ float* to = X + r * ldw;
        for (int k = 0; k < SG; k += 64)
          if (k + lane < SG) {
            global_to_lds(s0 + 4 * k, to + 4 * k);
            if (BR) global_to_lds(s1 + 4 * k, to + t.segp + 4 * k);
          }
      }
    }
    // the children's c of this thread's first forward (message, unit) pair
    float pcl = 0.f, pcr = 0.f;
    if (BR && (int)threadIdx.x < nF * nu) {
      const int r = by_nu(threadIdx.x), u = u0 + (int)threadIdx.x - r * nu;
      pcl = xbase[M.off0[r] + Hp + u];
      pcr = xbase[M.off1[r] + Hp + u];
    }
    asm volatile("" ::: "memory");   // all of these are on their way before anything below waits
    if (OPT == 2 && !formed) {
      pw1 *= (double)ob.b1;
      pw2 *= (double)ob.b2;
      c1 = uni((float)(1.0 / (1.0 - pw1)));
      c2 = uni((float)(1.0 / (1.0 - pw2)));
      formed = true;
    }
    for (int p = threadIdx.x; p < nB * nu; p += AMP_THREADS) {
      const int k = by_nu(p), j = p - k * nu;
      TreeDelta<BR, 18> d;
      d.fetch(B, M, nF + k, u0 + j, xbase);
      d.form(B, M, nF + k, j, nu, u0 + j, Y + (nF + k) * ldy);
    }
    for (int p = threadIdx.x; p < nB * (t.Rp - R); p += AMP_THREADS) {
      const int k = p / (t.Rp - R);
      Y[(nF + k) * ldy + R + p - k * (t.Rp - R)] = 0.f;
    }
    wait_vm();   // this wave's rows are in LDS
    lds_barrier();
    PHASE(0);
    // ---------------- products
    // (Splitting the columns of few forward messages over several items, whose sums then met in LDS, was taken out: evaluation at
    // hidden 37 5.53 -> 5.08 ms per 400 trees without it, at 80 7.45 -> 7.06, at 150 8.08 -> 8.00; only one tree at a time at 150 gains
    // from it, 9.85 -> 9.74 per 100.)
    {
      // gradient: G[r][c] += sum_k delta_k[r] x_k[c], k in ring order
      if (nB > 0 && unit_of(0) >= 0) {
        float a0[GU], a1[GU];
        v4f x0[GU], x1[GU];
        // beyond the batch: a row of zeros meets the last message's input
        auto fetch = [&](int k0, float (&a)[GU], v4f (&x)[GU]) {
          const int k = k0 + q, r = nF + (k < nB ? k : nB - 1);
          const LDSQ float* yr = (k < nB ? Y + r * ldy : Z) + i;
          const LDSQ float* xr = X + r * ldw;
#pragma unroll
          for (int u = 0; u < GU; ++u) {
            a[u] = yr[arow[u]];
            x[u] = *(const LDSQ v4f*)(xr + xcol[u]);
          }
        };
        auto add = [&](float (&a)[GU], v4f (&x)[GU]) {
#pragma unroll
          for (int u = 0; u < GU; ++u)
            if (wave * GU + u < NU) {
#pragma unroll
              for (int v = 0; v < 4; ++v) g[u][v] = MFMA(a[u], x[u][v], g[u][v]);
            }
        };
        fetch(0, a0, x0);
        for (int k0 = 0; k0 < nB; k0 += 8) {
          fetch(k0 + 4, a1, x1);
          add(a0, x0);
          if (k0 + 4 >= nB) break;
          fetch(k0 + 8, a0, x0);
          add(a1, x1);
        }
      }
      const int NBF = (nF + 15) >> 4, nFI = NRB * NBF, items = nFI + NCG * ((nB + 31) >> 5);
      auto next = [&]() {
        int it = 0;
        if (lane == 0) it = __hip_atomic_fetch_add((LDSQ int*)&s_item, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return it;
      };
      // this lane's messages of the input-gradient items: rows, and where their results go in either segment
      int rows_of = -1, j0 = 0;
      const LDSQ float *dr0 = Y, *dr1 = Y;
      GQ float *lo0 = obase, *lo1 = obase, *hi0 = obase, *hi1 = obase;
      int ahead = next();
      for (int it = uni(ahead); it < items; it = uni(ahead)) {
        ahead = next();
        if (it < nFI) {
          // Y[j][r] = b[r] + sum_c W[r][c] x_j[c]
          const int nb = by_nrb(it), rb = it - nb * NRB, j = nb * 16 + i;
          const LDSQ float* wp = Wl + (rb * 16 + i) * ldw + 4 * q;
          const LDSQ float* xp = X + (j < nF ? j : nF - 1) * ldw + 4 * q;
          v4f acc[4] = {*(const LDSQ v4f*)(bl + rb * 16 + 4 * q), zero, zero, zero};
          cell_rows(wp, xp, NCG, acc);
          if (j < nF) *(LDSQ v4f*)(Y + j * ldy + rb * 16 + 4 * q) = (acc[0] + acc[1]) + (acc[2] + acc[3]);
        } else {
          // dx_j[c] = sum_r W[r][c] delta_j[r]: 16 columns for up to 32 messages, from the accumulators to HBM
          const int bi = it - nFI, pb = bi >= NCG ? 1 : 0, cb = bi - pb * NCG;
          if (pb != rows_of) {
            rows_of = pb;
            j0 = pb * 32 + i;
            const int r0 = nF + (j0 < nB ? j0 : nB - 1), r1 = nF + (j0 + 16 < nB ? j0 + 16 : nB - 1);
            dr0 = Y + r0 * ldy + 4 * q;
            dr1 = Y + r1 * ldy + 4 * q;
            lo0 = obase + M.dst0[r0] + 4 * q;
            lo1 = obase + M.dst0[r1] + 4 * q;
            hi0 = obase + M.dst1[r0] + 4 * q - t.segp;
            hi1 = obase + M.dst1[r1] + 4 * q - t.segp;
          }
          const LDSQ float* wp = Wl + 4 * q * ldw + cb * 16 + i;
          v4f dx[2];
          if (pb * 32 + 16 < nB)
            cell_cols<2>(wp, ldw, dr0, dr1, NRB, dx);
          else
            cell_cols<1>(wp, ldw, dr0, dr1, NRB, dx);
          const int lc = cb * 16 + 4 * q;
          const bool hi = BR && lc >= t.segp;
          if (lc < t.Cl && j0 < nB) *(GQ v4f*)((hi ? hi0 : lo0) + cb * 16) = dx[0];
          if (lc < t.Cl && j0 + 16 < nB) *(GQ v4f*)((hi ? hi1 : lo1) + cb * 16) = dx[1];
        }
      }
    }
    PHASE(1);
    // ---------------- outputs
    if (nF > 0) {
      lds_barrier();
      for (int p = threadIdx.x; p < nF * nu; p += AMP_THREADS) {
        const int r = by_nu(p), j = p - r * nu, u = u0 + j;
        const bool first = p == (int)threadIdx.x;
        const float cl = BR ? (first ? pcl : xbase[M.off0[r] + Hp + u]) : 0.f;
        const float cr = BR ? (first ? pcr : xbase[M.off1[r] + Hp + u]) : 0.f;
        tree_activate<BR>(B, B.node(M.s[r], M.n[r]), Y + r * ldy, j, nu, u, cl, cr, wr.train);
      }
    }
    PHASE(2);
    // what lane r of wave 0 needs of row r for its joins, before the batch's record is given up
    const TreePost tp = tree_post_of(M, lane < n ? lane : 0, lane < n, lane < nF);
    // every wave's HBM stores have landed before wave 0 publishes the batch
    publish_barrier();
    PHASE(3);
    count += nB;
    const bool due = (int)count >= nd_muf;
    if (wave == 0) {
      fence_release();
      tree_publish<BR>(wr, B, tp);
    }
    PHASE(4);
    if (wave == 1) {
      // recorded by the wave that records the next batch's events, so that the update comes first
      if (due && lane == 0) log_event(D, W, &s_logn, wr.node, 2, 0, 0);
      take_batch(due ? 0u : count);
    }
    PHASE(5);
    // the bias gradient
    if (nB > 0 && brow >= 0) {
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int r = brow + a * BS;
        if (r < R) {
          const LDSQ float* yr = Y + nF * ldy + r;
          int k = 0;
          for (; k + 7 < nB; k += 8) {   // eight messages' deltas are read together; the sum keeps their order
            float y[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) y[b] = yr[(k + b) * ldy];
#pragma unroll
            for (int b = 0; b < 8; ++b) gb[a] += y[b];
          }
          for (; k < nB; ++k) gb[a] += yr[k * ldy];
        }
      }
    }
    PHASE(6);
    if (due) {
      // ---------------- the node's own update (Section 3): the optimizer's step on the weights in LDS
      tstep++;
      if (threadIdx.x == 0) note_update(D);
      OptCoef o = ob;
      o.kind = OPT;
      if (OPT == 2) {
        o.c1 = c1;
        o.c2 = c2;
        formed = false;
      }
      const float inv = uni(s_opt.mean) ? 1.f / (float)count : 1.f;
      if (unit_of(0) >= 0) {
#pragma unroll
        for (int u = 0; u < GU; ++u) {
          const int id = unit_of(u);
          if (id < 0) continue;   // lanes beyond the row rewrite its padding: their gradient is zero
          LDSQ float* wp = Wl + (arow[u] + 4 * q) * ldw + xcol[u];
          v4f m4[4], v4[4] = {zero, zero, zero, zero};
          if (!KEEP && OPT != 0) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int p = ((valid[u] >> (4 * v + e)) & 1u) ? at(u, v, e) : 0;
                m4[v][e] = ndM[p];
                v4[v][e] = OPT == 2 ? ndV[p] : 0.f;
              }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v4f w = *(LDSQ v4f*)(wp + e * ldw);
            if (OPT == 0) {
              // rows and columns of the padding have no gradient
              w -= (o.lr * inv) * (v4f){g[u][0][e], g[u][1][e], g[u][2][e], g[u][3][e]};
            } else {
              // (without a branch for each element: a padding one has no gradient and no slots either, and stays zero)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const bool real = (valid[u] >> (4 * v + e)) & 1u;
                float m = KEEP ? sm[KEEP ? u : 0][v][e] : real ? m4[v][e] : 0.f;
                float s = KEEP ? (OPT == 2 ? sv[KEEP && OPT == 2 ? u : 0][v][e] : 0.f) : real ? v4[v][e] : 0.f;
                w[v] = opt_step(o, w[v], g[u][v][e] * inv, m, s);
                if (KEEP) {
                  sm[KEEP ? u : 0][v][e] = m;
                  if (OPT == 2) sv[KEEP && OPT == 2 ? u : 0][v][e] = s;
                } else if (real) {
                  const int p = at(u, v, e);
                  ndM[p] = m;
                  if (OPT == 2) ndV[p] = s;
                }
              }
            }
            *(LDSQ v4f*)(wp + e * ldw) = w;
          }
          if (OPT == 2 && ob.eps == 0.f)   // but for 0 / 0
            for (int k = 0; k < 16; ++k)
              if (!((valid[u] >> k) & 1u)) wp[(k & 3) * ldw + (k >> 2)] = 0.f;
#pragma unroll
          for (int v = 0; v < 4; ++v) g[u][v] = zero;
        }
      }
      if (brow >= 0 && nd.has_bias) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const int r = brow + a * BS;
          if (r < R) bl[r] = opt_step(o, bl[r], gb[a] * inv, bm[a], bv[a]);
          gb[a] = 0.f;
        }
      }
      count = 0;
    }
    lds_barrier();
    PHASE(7);
  }
  tile_store(nd, t, Wg, bg);
#pragma unroll
  for (int u = 0; u < GU; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((valid[u] >> (4 * v + e)) & 1u) {
          const int p = at(u, v, e);
          if (count > 0) ndG[p] = g[u][v][e];
          if (KEEP && slots) ndM[p] = sm[KEEP ? u : 0][v][e];
          if (KEEP && OPT == 2 && slots) ndV[p] = sv[KEEP && OPT == 2 ? u : 0][v][e];
        }
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int r = brow + a * BS;
    if (brow >= 0 && r < R && nd.has_bias) {
      const int p = nd.rows * t.C + rowmap[r];
      if (count > 0) ndG[p] = gb[a];
      if (slots) ndM[p] = bm[a];
      if (slots && OPT == 2) ndV[p] = bv[a];
    }
  }
  if (threadIdx.x == 0) {
    W->wstate[0] = count;
    W->wstate[1] = tstep;
  }
}
