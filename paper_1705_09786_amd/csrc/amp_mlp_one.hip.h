// The whole MLP on one compute unit: its three layers, the loss and the controller are the work of worker 0's workgroup, and
// the layers' own workgroups leave at once (mlp_one_fits says when).
//
// What bounds it: an instance visits five stages behind each other and a stage is one small matrix-vector product, so between
// workgroups (role_mlp_regs) nearly all of its time is hand-overs -- poll, fetch, product, drain, post.  Here a stage ends at a
// workgroup barrier and its result is in LDS, and up to four instances at a time (the messages a 4x4x1 matrix instruction
// takes) go through a stage together.  Measured, 64-128-128-10 with an update per gradient: 1,024 instances with four in
// flight 3.54 -> 1.18 ms, 4.4 us a group, of which a wave's 454 matrix instructions (8 cycles each and 8.4 from one to the
// next) are 1.6; a call on eight instances one at a time 124 -> 90 us.  Evaluation of a small model 2.07 -> 0.42 ms.
//   * Weights stay in registers, once with an output per lane (forward) and, where a gradient goes on to the layer below, once
//     with an input per lane (backward); one wave to a SIMD has 512 registers a lane.  Operands are the instances' values from
//     LDS, broadcast to the sixteen blocks of the instruction; the four waves split outputs and contraction, their parts meet in
//     LDS and the next stage adds them up while it reads them.
//   * A plain SGD step is the same instruction: weights += (-lr delta) (x) input accumulates into the weights themselves, in
//     both layouts with the same rounding.
//   * With an update per gradient, message m's backward pass meets weights that the messages before it have just changed:
//     W_m^T d_m = W_0^T d_m - lr sum_{j < m} x_j (d_j . d_m).  So the products of all messages are formed at once from the
//     weights before the group and corrected by the dot products of their deltas, instead of one behind the other.
// The event order is that of a node which takes the group's forward messages, then its backward ones, an update behind each (or
// behind the one that completes min_update_frequency: a group never reaches past an update otherwise).
#pragma once
#include <type_traits>

// acc[e] += A[4 block + e] * B[lane]: A is block ABID's four values, broadcast to all sixteen blocks.
#define MFMA4(a, b, c, abid) __builtin_amdgcn_mfma_f32_4x4x1f32((a), (b), (c), 4, (abid), 0)
#define MO_LD 144   // row stride of [message][unit] arrays: 16 modulo the 64 banks, so that four messages' reads spread
#define MO_LT 132   // row stride of a layer's tile: rows 16-byte aligned and spread over the banks

// Plain SGD at layers of up to 128 x 128, and every evaluation of such layers.  Gradients that wait for an update take as many
// registers as the weights: with more than 64 inputs and more than 64 hidden units that is more than there are.  With more than 64
// hidden units alone the line is at four gradients an update, where it was drawn when the loop with waiting gradients spilled
// (an update every 3 then took as long on one workgroup as on three).  It no longer does, and equal thresholds of 2 and 3 would
// gain as well; unequal ones as small cut the groups to one or two instances.  512 instances of 64-128-128-10, a workgroup per
// layer / here, with one, two and four in flight: an update every 2 4.13 / 2.53 ms, 2.57 / 1.65, 2.09 / 1.64; every 3 4.12 / 2.33, 2.52 /
// 1.74, 2.06 / 1.15; every 4 4.15 / 2.24, 2.55 / 1.34, 2.05 / 0.89; every 8 4.15 / 2.10, 2.53 / 1.19, 2.03 / 0.74; 64 hidden units
// every 2 4.11 / 1.98, 2.54 / 1.25, 2.06 / 1.25.  The same in every workgroup of the replica.
__device__ __forceinline__ bool mlp_one_each(const GQ AmpDev* D) {   // no gradient ever waits
  bool each = true;
#pragma unroll
  for (int l = 0; l < 3; ++l) each = each && D->node[l].muf == 1 && D->worker[1 + l].wstate[0] == 0u;
  return each || !D->train;
}
__device__ __forceinline__ bool mlp_one_fits(const GQ AmpDev* D) {
  if (D->hidden > MLP_MAX || D->d_in > MLP_MAX || D->n_class > 64) return false;
  if (!D->train) return true;
  if (D->node[0].opt != 0 || D->node[1].opt != 0 || D->node[2].opt != 0) return false;
  if (D->hidden <= 64 || mlp_one_each(D)) return true;
  return D->d_in <= 64 && D->node[0].muf >= 4 && D->node[1].muf >= 4 && D->node[2].muf >= 4;
}

// A wave's share of a product: 64 outputs, one a lane, from out0 on, and NJ groups of 16 terms from k0 on.  The SPLITS waves that
// share the outputs each leave a part.  What lies beyond the layer is zero.
template <int SPLITS, int NJ>
struct MoPiece {
  int out0, k0, part;
  __device__ __forceinline__ explicit MoPiece(int wave) : out0(64 * (wave / SPLITS)), k0(16 * NJ * (wave % SPLITS)), part(wave % SPLITS) {}
};

// Four messages against the wave's piece: sum_k w[k] x_m[k] for message m = 0..3 in component m.  xv[j] of lane l holds
// x[message l % 4][16 j + l / 4].  Spelt out, with the waits that its operands and its result need: weights that are accumulated
// into lie in the accumulation registers (R "a"), from where the instruction can take them as they are, but the compiler copies
// every one of them out first (230 moves per group of messages, 0.4 us).
#define MO_M(d, w, c, id) "v_mfma_f32_4x4x1_16b_f32 " d ", %4, " w ", " c " cbsz:4 abid:" #id "\n\t"
#define MO_M12 \
  MO_M("%0", "%9", "%0", 4) MO_M("%1", "%10", "%1", 5) MO_M("%2", "%11", "%2", 6) MO_M("%3", "%12", "%3", 7) \
  MO_M("%0", "%13", "%0", 8) MO_M("%1", "%14", "%1", 9) MO_M("%2", "%15", "%2", 10) MO_M("%3", "%16", "%3", 11) \
  MO_M("%0", "%17", "%0", 12) MO_M("%1", "%18", "%1", 13) MO_M("%2", "%19", "%2", 14) MO_M("%3", "%20", "%3", 15)
#define MO_Q(R, q) R(q[0]), R(q[1]), R(q[2]), R(q[3])
#define MO_DOT(R)                                                                                                                   \
  asm volatile("s_nop 1\n\t" MO_M("%0", "%5", "0", 0) MO_M("%1", "%6", "0", 1) MO_M("%2", "%7", "0", 2) MO_M("%3", "%8", "0", 3)     \
                   MO_M12 "s_nop 5"                                                                                                 \
               : "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3)                                                                         \
               : "v"(xv[0]), MO_Q(R, w[0]), MO_Q(R, w[1]), MO_Q(R, w[2]), MO_Q(R, w[3]));                                           \
  _Pragma("unroll") for (int j = 1; j < NJ; ++j)                                                                                    \
    asm volatile("s_nop 1\n\t" MO_M("%0", "%5", "%0", 0) MO_M("%1", "%6", "%1", 1) MO_M("%2", "%7", "%2", 2)                        \
                     MO_M("%3", "%8", "%3", 3) MO_M12 "s_nop 5"                                                                     \
                 : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3)                                                                           \
                 : "v"(xv[j]), MO_Q(R, w[4 * j]), MO_Q(R, w[4 * j + 1]), MO_Q(R, w[4 * j + 2]), MO_Q(R, w[4 * j + 3]));
template <bool ACC, int NJ>   // ACC: the weights are in the accumulation registers
__device__ __forceinline__ v4f mo_dot(const v4f (&w)[4 * NJ], const float (&xv)[NJ]) {
  v4f a0, a1, a2, a3;
  if constexpr (ACC) {
    MO_DOT("a")
  } else {
    MO_DOT("v")
  }
  return (a0 + a1) + (a2 + a3);
}
// w[k] += a(lane k) * b(this lane)
#define MO_ADD(g) w[g] = MFMA4(a, b, w[g], g);
#define MO_ADD16(j) \
  if constexpr ((j) < NJ) { MO_ADD(4 * (j)) MO_ADD(4 * (j) + 1) MO_ADD(4 * (j) + 2) MO_ADD(4 * (j) + 3) }
template <int NJ4>
__device__ __forceinline__ void mo_add(v4f (&w)[NJ4], float a, float b) {
  constexpr int NJ = NJ4 / 4;
  MO_ADD16(0) MO_ADD16(1) MO_ADD16(2) MO_ADD16(3)
}
// The same with w in the architectural registers: the builtin accumulates into the other half of the register file alone, and the
// five pieces of a wave are more than that half holds.  (Spelt out, so the waits a result needs before anything else may read it
// stand here as well.)
#define MO_ASM4(j, x0, x1, x2, x3)                                                                                                \
  if constexpr ((j) < NJ) {                                                                                                       \
    asm volatile("s_nop 4\n\tv_mfma_f32_4x4x1_16b_f32 %0, %4, %5, %0 cbsz:4 abid:" #x0                                           \
                 "\n\tv_mfma_f32_4x4x1_16b_f32 %1, %4, %5, %1 cbsz:4 abid:" #x1                                                  \
                 "\n\tv_mfma_f32_4x4x1_16b_f32 %2, %4, %5, %2 cbsz:4 abid:" #x2                                                  \
                 "\n\tv_mfma_f32_4x4x1_16b_f32 %3, %4, %5, %3 cbsz:4 abid:" #x3 "\n\ts_nop 7\n\ts_nop 1"                         \
                 : "+v"(w[4 * (j)]), "+v"(w[4 * (j) + 1]), "+v"(w[4 * (j) + 2]), "+v"(w[4 * (j) + 3])                             \
                 : "v"(a), "v"(b));                                                                                               \
  }
template <int NJ4>
__device__ __forceinline__ void mo_add_v(v4f (&w)[NJ4], float a, float b) {
  constexpr int NJ = NJ4 / 4;
  MO_ASM4(0, 0, 1, 2, 3)
  MO_ASM4(1, 4, 5, 6, 7)
  MO_ASM4(2, 8, 9, 10, 11)
  MO_ASM4(3, 12, 13, 14, 15)
}

// The dot products of four messages' values (laid out as for mo_dot): those of message v with message l in component v of lane l.
template <int NJ>
__device__ __forceinline__ v4f mo_gram(const float (&xv)[NJ]) {
  v4f g = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < NJ; ++j) g = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[j], xv[j], g, 0, 0, 0);
#pragma unroll
  for (int v = 0; v < 3; ++v) {   // the last message's are not asked for
    float s = g[v];
    s += dpp<DPP_ROR8>(s);
    s += dpp<DPP_ROR4>(s);
    s = swap_add16(s, s);
    g[v] = swap_add32(s, s);
  }
  return g;
}

// A layer's rows, C <= 128 floats each, between memory and an LDS tile of OUT rows, zero beyond the layer.
template <int OUT>
__device__ __forceinline__ void mo_tile_load(LDSQ float* T, const GQ float* P, int R, int C) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int r0 = wave; r0 < OUT; r0 += 32) {
    float v[8][2];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = r0 + 4 * u, c = lane + 64 * h;
        const bool in = r < R && c < C;
        const float x = P[in ? r * C + c : 0];
        v[u][h] = in ? x : 0.f;
      }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) T[(r0 + 4 * u) * MO_LT + lane + 64 * h] = v[u][h];
  }
}
__device__ __forceinline__ void mo_tile_store(const LDSQ float* T, GQ float* P, int R, int C) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int r = wave; r < R; r += 4)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (lane + 64 * h < C) P[r * C + lane + 64 * h] = T[r * MO_LT + lane + 64 * h];
}
// A wave's piece from the tile and back: a row of the layer to a lane, or a column.
template <int SPLITS, int NJ>
__device__ __forceinline__ void mo_rows(const LDSQ float* T, v4f (&w)[4 * NJ], const MoPiece<SPLITS, NJ>& p) {
  const LDSQ float* t = T + (p.out0 + (threadIdx.x & 63)) * MO_LT + p.k0;
#pragma unroll
  for (int g = 0; g < 4 * NJ; ++g) w[g] = *(const LDSQ v4f*)(t + 4 * g);
}
template <int SPLITS, int NJ>
__device__ __forceinline__ void mo_rows_back(LDSQ float* T, const v4f (&w)[4 * NJ], const MoPiece<SPLITS, NJ>& p) {
  LDSQ float* t = T + (p.out0 + (threadIdx.x & 63)) * MO_LT + p.k0;
#pragma unroll
  for (int g = 0; g < 4 * NJ; ++g) *(LDSQ v4f*)(t + 4 * g) = w[g];
}
template <int SPLITS, int NJ>
__device__ __forceinline__ void mo_cols(const LDSQ float* T, v4f (&w)[4 * NJ], const MoPiece<SPLITS, NJ>& q) {
  const LDSQ float* t = T + q.k0 * MO_LT + q.out0 + (threadIdx.x & 63);
#pragma unroll
  for (int g = 0; g < 4 * NJ; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e) w[g][e] = t[(4 * g + e) * MO_LT];
}

// Weights as they are, in groups of four registers: otherwise the compiler carries them round the loop one by one, in
// registers of its choice, and moves them all.
template <bool ACC, int N>
__device__ __forceinline__ void mo_keep(v4f (&w)[N]) {
#pragma unroll
  for (int g = 0; g < N; ++g) {
    if constexpr (ACC)
      asm volatile("" : "+a"(w[g]));
    else
      asm volatile("" : "+v"(w[g]));
  }
}

__shared__ unsigned s_mo_logn[3];
__shared__ int s_mo_full;   // a record is full: of the threads that write them alone

// An event of layer l, in its own worker's record.  ONE thread.
__device__ __forceinline__ void mo_log(const GQ AmpDev* D, int l, int kind, unsigned seq) {
  const GQ WorkerDev& w = D->worker[1 + l];
  const unsigned n = s_mo_logn[l];
  if (n >= w.log_cap) {
    raise_abort(D, ABORT_LOG_FULL, 1 + l);
    s_mo_full = 1;
    return;
  }
  ((GQ unsigned long long*)w.log)[n] = ((unsigned long long)seq << 32) | ((unsigned)kind << 28) | ((unsigned)l << 20);
  s_mo_logn[l] = n + 1;
}
// The same of the controller.
__device__ __forceinline__ void mo_log_ctrl(const GQ AmpDev* D, const GQ WorkerDev* W, int kind, unsigned seq, unsigned local) {
  if (s_logn >= s_log_cap) s_mo_full = 1;
  log_event(D, W, &s_logn, 0, kind, seq, local);
}

// The controller's books, kept by ONE wave and only where somebody asks: a bounded limit, or the record.  (As scalars of every
// wave they cost the loop registers it does not have: 1,024 instances 1.21 -> 1.26 ms.)  What a group's events, its
// retirements and the admissions behind them come to is known as it begins, so that wave settles it beside the loss layer.
struct alignas(16) MoAdmission {
  int limit, flying, most;   // in flight at most / now / at most so far
  int full;                  // s_mo_full as the group begins: every wave leaves in front of the same one
  int mak, in, out;          // places of the next admission and the next retirement in upd_at, which has max_active_keys of them
  unsigned admitted;
  float bound, per_worker;   // (no bound: one that nothing reaches)
};
__shared__ MoAdmission s_mo_adm;

// A group's n <= 4 instances retire -- lane m's when `then` updates have been applied -- and others are admitted behind `after`, by the
// policies of role_ctrl: what is in flight and not in a group waits in front of the first layer.  done: retired with this group;
// upd_at: updates applied before each admission in flight.
__device__ __forceinline__ void mo_settle(const GQ AmpDev* D, const GQ WorkerDev* W, int lane, LDSQ unsigned* upd_at, unsigned n_total,
                                          unsigned done, int n, unsigned then, unsigned after) {
  MoAdmission A = s_mo_adm;
  const int full = s_mo_full, at = A.out + (lane < n ? lane : 0);
  const float seen = (float)(then - upd_at[at < A.mak ? at : at - A.mak]) * A.per_worker;
  const unsigned over = (unsigned)__ballot(seen > A.bound);
#pragma unroll
  for (int m = 0; m < 4; ++m)
    if (m < n) {
      A.limit += (over >> m) & 1u ? -1 : 1;
      A.limit = A.limit < 1 ? 1 : A.limit > A.mak ? A.mak : A.limit;
    }
  A.out = A.out + n < A.mak ? A.out + n : A.out + n - A.mak;
  const unsigned left = n_total - A.admitted;
  A.flying = (int)(A.admitted - done);
  int more = A.limit - A.flying;
  more = more < 0 ? 0 : (unsigned)more < left ? more : (int)left;
  for (int i = lane; i < more; i += 64) upd_at[A.in + i < A.mak ? A.in + i : A.in + i - A.mak] = after;
  if (s_log_cap && lane == 0)
    for (unsigned i = A.admitted; i < A.admitted + (unsigned)more; ++i)
      mo_log_ctrl(D, W, 3, s_first_seq + i, D->adm_inst && D->adm_inst[i] < 0 ? 1u : 0u);
  A.in = A.in + more < A.mak ? A.in + more : A.in + more - A.mak;
  A.full = full;
  A.admitted += (unsigned)more;
  A.flying += more;
  if (A.flying > A.most) A.most = A.flying;
  if (lane == 0) s_mo_adm = A;
}

// EACH: an update per gradient at every layer (and every evaluation): no gradient is kept.  BIG: more than 64 hidden units, two
// pieces of outputs.  NJ1: groups of 16 inputs a wave takes in the first layer.
template <bool EACH, bool BIG, int NJ1>
__device__ __forceinline__ void role_mlp_one(const GQ AmpDev* D, const GQ WorkerDev* W) {
  // The accumulation registers, half of the file, take what is accumulated into -- the weights under EACH, all five pieces where
  // they fit, otherwise the gradients -- and the transposed pieces; the rest is in the other half.
  constexpr bool ACC = EACH, VACC = !EACH || !BIG || NJ1 < 4;
  constexpr int SP = BIG ? 2 : 4, NJ2 = BIG ? 4 : 1, NJ3 = BIG ? 2 : 1, OUT = BIG ? 128 : 64;
  const int H = uni(D->hidden), C1 = uni(D->d_in), K = uni(D->n_class), train = uni(D->train);
  const int wave = uni((int)(threadIdx.x >> 6));
  const MoPiece<SP, NJ1> p1(wave);
  const MoPiece<SP, NJ2> p2(wave);   // of the second layer and of its transpose
  const MoPiece<4, NJ3> p3(wave);
  const MoPiece<SP, NJ3> q3(wave);
  Lds L{amp_lds};
  LDSQ float* T = (LDSQ float*)L.take(MLP_MAX * MO_LT);   // a layer on its way to the other layout
  LDSQ float* T1 = (LDSQ float*)L.take(0);                // a second tile, at the start and the end; between them:
  LDSQ float* P1 = (LDSQ float*)L.take(16 * MO_LD);       // parts of the stages' products, [part][message][unit]
  LDSQ float* P2 = (LDSQ float*)L.take(16 * MO_LD);
  LDSQ float* P3 = (LDSQ float*)L.take(16 * MO_LD);
  LDSQ float* P4 = (LDSQ float*)L.take(16 * MO_LD);
  LDSQ float* P5 = (LDSQ float*)L.take(16 * MO_LD);
  LDSQ float* X = (LDSQ float*)L.take(2 * 4 * MO_LD);     // inputs (two groups'), activations, deltas, [message][unit]
  LDSQ float* H1 = (LDSQ float*)L.take(4 * MO_LD);
  LDSQ float* H2 = (LDSQ float*)L.take(4 * MO_LD);
  LDSQ float* DZ = (LDSQ float*)L.take(4 * MO_LD);
  LDSQ float* D2 = (LDSQ float*)L.take(4 * MO_LD);
  L.take(MLP_MAX * MO_LT - (5 * 16 + 2 * 4 + 4 * 4) * MO_LD);
  LDSQ float* b1 = (LDSQ float*)L.take(MO_LD);
  LDSQ float* b2 = (LDSQ float*)L.take(MO_LD);
  LDSQ float* b3 = (LDSQ float*)L.take(MO_LD);
  LDSQ unsigned* upd_at = (LDSQ unsigned*)L.take(AMP_MAX_MAK);
  const float lr1 = uni(D->node[0].lr), lr2 = uni(D->node[1].lr), lr3 = uni(D->node[2].lr);
  unsigned c1 = uni(D->worker[1].wstate[0]), c2 = uni(D->worker[2].wstate[0]), c3 = uni(D->worker[3].wstate[0]);
  unsigned u1 = 0, u2 = 0, u3 = 0;   // the layers' updates, where gradients wait; else one for every gradient
  const long long t_begin = wall_clock64();
  // ---- weights: rows of every layer (an output per lane), columns of the upper two
  v4f w1[4 * NJ1], w2[4 * NJ2], v2[4 * NJ2], w3[4 * NJ3], v3[4 * NJ3];
  v4f g1[EACH ? 4 : 4 * NJ1], g2[EACH ? 4 : 4 * NJ2], g3[EACH ? 4 : 4 * NJ3];
  float gb1 = 0.f, gb2 = 0.f, gb3 = 0.f;
  {
    const int tid = threadIdx.x;
    const GQ float *const W1 = uni_gq<float>(D->node[0].P), *const W2 = uni_gq<float>(D->node[1].P), *const W3 = uni_gq<float>(D->node[2].P);
    mo_tile_load<OUT>(T, W2, H, H);
    mo_tile_load<OUT>(T1, W1, H, C1);
    __syncthreads();
    mo_rows(T, w2, p2);
    mo_cols(T, v2, p2);
    mo_rows(T1, w1, p1);
    lds_barrier();
    mo_tile_load<64>(T, W3, K, H);
    for (int i = tid; i < MO_LD; i += AMP_THREADS) {
      b1[i] = i < H ? W1[H * C1 + i] : 0.f;
      b2[i] = i < H ? W2[H * H + i] : 0.f;
      b3[i] = i < K ? W3[K * H + i] : 0.f;
    }
    __syncthreads();
    mo_rows(T, w3, p3);
    mo_cols(T, v3, q3);
    if constexpr (!EACH) {
      const v4f zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int g = 0; g < 4 * NJ1; ++g) g1[g] = zero;
#pragma unroll
      for (int g = 0; g < 4 * NJ2; ++g) g2[g] = zero;
#pragma unroll
      for (int g = 0; g < 4 * NJ3; ++g) g3[g] = zero;
      // gradients carried over from the previous launch
      if (c1 | c2 | c3) {
        const GQ float *const G1 = uni_gq<float>(D->node[0].G), *const G2 = uni_gq<float>(D->node[1].G), *const G3 = uni_gq<float>(D->node[2].G);
        const int o1 = p1.out0 + (tid & 63);
        __syncthreads();
        mo_tile_load<OUT>(T, G1, H, C1);
        __syncthreads();
        mo_rows(T, g1, p1);
        __syncthreads();
        mo_tile_load<OUT>(T, G2, H, H);
        __syncthreads();
        mo_rows(T, g2, p2);
        __syncthreads();
        mo_tile_load<64>(T, G3, K, H);
        __syncthreads();
        mo_rows(T, g3, p3);
        gb1 = o1 < H ? G1[H * C1 + o1] : 0.f;
        gb2 = o1 < H ? G2[H * H + o1] : 0.f;
        gb3 = tid < K ? G3[K * H + tid] : 0.f;
      }
    }
  }
  const GQ float* datax = uni_gq<float>(D->data.x);
  const GQ int* lab = uni_gq<int>(D->data.lab);
  const GQ int* adm = uni_gq<int>(D->adm_inst);
  GQ float* loss_out = uni_gq<float>(D->loss_out);
  GQ int* correct_out = uni_gq<int>(D->correct_out);
  const unsigned n_total = uni(D->n_total), n_inst = (unsigned)uni(D->data.n_inst);
  const int four_at_most = uni(D->mak) < 4 ? uni(D->mak) : 4;
  const bool books = uni(D->admit_bounded) != 0 || uni(s_log_cap) != 0u;
  unsigned done = 0, groups = 0, trained_all = 0;
  auto updates = [&]() { return EACH ? 3u * trained_all : u1 + u2 + u3; };
  if (threadIdx.x < 3) s_mo_logn[threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    s_mo_full = 0;
    s_mo_adm = {D->admit_bounded ? 1 : D->mak, 0, 0, 0, D->mak, 0, 0, 0u, D->admit_bounded ? D->max_staleness : 3e38f, 1.f / (float)D->n_updaters};
  }
  // the instance word of the launch's admission `at` (sign bit: forward only), the last one's beyond it
  auto word_of = [&](unsigned at) -> int {
    if (at >= n_total) at = n_total - 1u;
    return adm ? adm[at] : (int)(at % n_inst);
  };
  // the next group's inputs, as the first layer's operand, and label: lane l for message l % 4
  float xn[NJ1];
  int word = 0, label = 0;
  auto fetch = [&](int lane) {
    const int inst = word & 0x7fffffff, k0 = p1.k0 + (lane >> 2);
    const GQ float* x = datax + (long long)inst * C1;
#pragma unroll
    for (int j = 0; j < NJ1; ++j) {
      const int k = k0 + 16 * j;
      const float v = x[k < C1 ? k : 0];
      xn[j] = k < C1 ? v : 0.f;
    }
    label = lab[inst];   // one label per instance
  };
  if (threadIdx.x == 0) D->clock[0] = wall_clock64();
  if (books) {
    __syncthreads();
    if (wave == 3) mo_settle(D, W, threadIdx.x & 63, upd_at, n_total, 0u, 0, 0u, 0u);
  }
  word = word_of(threadIdx.x & 3u);
  fetch(threadIdx.x & 63);
  __syncthreads();
  while (done < n_total) {
    mo_keep<ACC>(w1);
    mo_keep<ACC>(w2);
    mo_keep<ACC>(w3);
    mo_keep<VACC>(v2);
    mo_keep<true>(v3);
    if constexpr (!EACH) {
      mo_keep<true>(g1);
      mo_keep<true>(g2);
      mo_keep<true>(g3);
    }
    // what follows from the thread's index is computed anew for every group: as loop invariants these values would be spilled
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, m4 = lane & 3, k4 = lane >> 2, o1 = p1.out0 + lane;
    const int mrow = m4 * MO_LD + k4;   // where an operand of this lane lies in a [message][unit] array, from its first term on
    // ---------------- admission
    int n = four_at_most;
    if (books) {
      if (uni(s_mo_adm.full)) break;
      const int flying = uni(s_mo_adm.flying);
      n = flying < 4 ? flying : 4;
    }
    if ((unsigned)n > n_total - done) n = (int)(n_total - done);
    if (!EACH) {
      const int r1 = uni(D->node[0].muf) - (int)c1, r2 = uni(D->node[1].muf) - (int)c2, r3 = uni(D->node[2].muf) - (int)c3;
      int room = r1 < r2 ? r1 : r2;
      room = r3 < room ? r3 : room;
      if (room < 1) room = 1;   // a threshold lowered between two calls
      if (n > room) n = room;
    }
    const unsigned tr = train ? ~(unsigned)__ballot(word < 0) & ((1u << n) - 1u) : 0u;   // those that train
    const int nt = __popc(tr), lab_now = label;
    groups++;
    auto put = [&](LDSQ float* P, int part, int out0, v4f r) {
#pragma unroll
      for (int e = 0; e < 4; ++e) P[(part * 4 + e) * MO_LD + out0 + lane] = r[e];
    };
    // the sum over the parts at `at` = message * MO_LD + unit
    auto sum = [&](const LDSQ float* P, auto parts, int at) {
      float s = P[at];
#pragma unroll
      for (int p = 1; p < decltype(parts)::value; ++p) s += P[p * 4 * MO_LD + at];
      return s;
    };
    constexpr std::integral_constant<int, SP> sp{};
    constexpr std::integral_constant<int, 4> four{};
    // ---------------- forward, layer 1
    LDSQ float* Xg = X + (groups & 1u) * 4 * MO_LD;
    {
      float xv[NJ1];
#pragma unroll
      for (int j = 0; j < NJ1; ++j) {
        xv[j] = m4 < n ? xn[j] : 0.f;
        if (p1.out0 == 0) Xg[mrow + p1.k0 + 16 * j] = xv[j];
      }
      put(P1, p1.part, p1.out0, mo_dot<ACC>(w1, xv));
    }
    word = word_of(done + (unsigned)(n + m4));   // on its way
    lds_barrier();
    PHASE(0);
    // ---------------- layer 2
    {
      float xv[NJ2];
#pragma unroll
      for (int j = 0; j < NJ2; ++j) xv[j] = fmaxf(sum(P1, sp, mrow + p2.k0 + 16 * j) + b1[p2.k0 + 16 * j + k4], 0.f);
      if (p2.out0 == 0)
#pragma unroll
        for (int j = 0; j < NJ2; ++j) H1[mrow + p2.k0 + 16 * j] = xv[j];
      put(P2, p2.part, p2.out0, mo_dot<ACC>(w2, xv));
    }
    lds_barrier();
    PHASE(1);
    // ---------------- layer 3
    {
      float xv[NJ3];
#pragma unroll
      for (int j = 0; j < NJ3; ++j) xv[j] = fmaxf(sum(P2, sp, mrow + p3.k0 + 16 * j) + b2[p3.k0 + 16 * j + k4], 0.f);
#pragma unroll
      for (int j = 0; j < NJ3; ++j) H2[mrow + p3.k0 + 16 * j] = xv[j];
      put(P3, p3.part, 0, mo_dot<ACC>(w3, xv));
    }
    fetch(lane);   // the next group's inputs arrive behind the rest of this one
    lds_barrier();
    PHASE(2);
    // ---------------- softmax cross-entropy: a wave per message, lane k = class k
    {
      const int lb = __builtin_amdgcn_readlane(lab_now, wave);
      const float zs = sum(P3, four, wave * MO_LD + lane) + b3[lane];
      const float z = lane < K ? zs : -3.0e38f;
      const float mx = wave_max(z);
      const float e = lane < K ? expf(z - mx) : 0.f;
      const float se = wave_sum(e);
      DZ[wave * MO_LD + lane] = ((tr >> wave) & 1u) && lane < K ? e / se - (lane == lb ? 1.f : 0.f) : 0.f;
      if (wave < n) {
        const unsigned long long top = __ballot(lane < K && z == mx);   // none where every logit is NaN
        const int best = top ? __builtin_ctzll(top) : 0;   // the first class with the largest logit
        const float zl = lane_of(z, lb);
        if (lane == 0) {
          loss_out[done + (unsigned)wave] = -(zl - mx - logf(se));
          correct_out[done + (unsigned)wave] = best == lb;
        }
      }
    }
    if (books && wave == 3) {   // the group retires -- a message behind the updates it brings about -- and others are admitted
      unsigned after = updates() + 3u * (unsigned)nt, mine = updates() + 3u * (unsigned)__popc(tr & ((2u << m4) - 1u));
      if constexpr (!EACH) {
        auto due = [&](int l, unsigned c) { return nt && (int)c + nt >= uni(D->node[l].muf) ? 1u : 0u; };
        after = updates() + due(0, c1) + due(1, c2) + due(2, c3);
        mine = m4 == n - 1 ? after : updates();
      }
      if (s_log_cap && lane == 0) {
        const unsigned seq0 = s_first_seq + done;
        for (int l = 0; l < 3; ++l) {
          for (int m = 0; m < n; ++m) mo_log(D, l, 0, seq0 + (unsigned)m);
          for (int m = 0; m < n; ++m)
            if ((tr >> m) & 1u) {
              mo_log(D, l, 1, seq0 + (unsigned)m);
              if (EACH) mo_log(D, l, 2, 0);
            }
        }
        for (int m = 0; m < n; ++m) mo_log_ctrl(D, W, 4, seq0 + (unsigned)m, 0);
      }
      mo_settle(D, W, lane, upd_at, n_total, done + (unsigned)n, n, mine, after);
    }
    lds_barrier();
    PHASE(3);
    if (tr) {
      // message m's product with the weights as the messages before it have left them
      auto follow = [&](v4f& r, const auto& d, float lr, const LDSQ float* in) {
        if (!EACH || nt < 2) return;
        float x[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) x[j] = in[j * MO_LD];
        const v4f g = mo_gram(d);
#pragma unroll
        for (int j = 0; j < 3; ++j)
          if ((tr >> j) & 1u) {
#pragma unroll
            for (int m = j + 1; m < 4; ++m)
              if ((tr >> m) & 1u) r[m] = fmaf(-lr * lane_of(g[j], m), x[j], r[m]);
          }
      };
      // ---------------- backward, layer 3
      {
        float xv[NJ3];
#pragma unroll
        for (int j = 0; j < NJ3; ++j) xv[j] = DZ[mrow + q3.k0 + 16 * j];
        v4f r = mo_dot<true>(v3, xv);
        follow(r, xv, lr3, H2 + q3.out0 + lane);
        put(P4, q3.part, q3.out0, r);
      }
      {
        float d[4], h[4], dk[4], ho[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          d[m] = DZ[m * MO_LD + lane];
          h[m] = H2[m * MO_LD + p3.k0 + lane];
          if (EACH) dk[m] = DZ[m * MO_LD + q3.k0 + lane];
          if (EACH) ho[m] = H2[m * MO_LD + q3.out0 + lane];
        }
        float b = b3[lane];
#pragma unroll
        for (int m = 0; m < 4; ++m)
          if ((tr >> m) & 1u) {
            if constexpr (EACH) {
              mo_add(w3, h[m], -lr3 * d[m]);
              mo_add(v3, -lr3 * dk[m], ho[m]);
              b = fmaf(-lr3, d[m], b);
            } else {
              mo_add(g3, h[m], d[m]);
              gb3 += d[m];
            }
          }
        if (EACH && wave == 0) b3[lane] = b;
      }
      lds_barrier();
      PHASE(4);
      // ---------------- layer 2
      {
        float xv[NJ2];
#pragma unroll
        for (int j = 0; j < NJ2; ++j) {
          const int at = mrow + p2.k0 + 16 * j;
          const float dh = sum(P4, sp, at);
          xv[j] = H2[at] > 0.f ? dh : 0.f;
        }
        if (p2.out0 == 0)
#pragma unroll
          for (int j = 0; j < NJ2; ++j) D2[mrow + p2.k0 + 16 * j] = xv[j];
        v4f r = mo_dot<VACC>(v2, xv);
        follow(r, xv, lr2, H1 + p2.out0 + lane);
        put(P5, p2.part, p2.out0, r);
      }
      lds_barrier();
      PHASE(5);
      // ---------------- layer 1's delta, the gradients of layers 1 and 2
      {
        float d1[4], d2[4], x[4], h[4], dk[4], ho[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const float s = sum(P5, sp, m * MO_LD + o1);
          ho[m] = H1[m * MO_LD + o1];
          d1[m] = ho[m] > 0.f ? s : 0.f;
          d2[m] = D2[m * MO_LD + o1];
          x[m] = Xg[m * MO_LD + p1.k0 + lane];
          h[m] = H1[m * MO_LD + p2.k0 + lane];
          if (EACH) dk[m] = D2[m * MO_LD + p2.k0 + lane];
        }
        float ba = b1[o1], bb = b2[o1];
#pragma unroll
        for (int m = 0; m < 4; ++m)
          if ((tr >> m) & 1u) {
            if constexpr (EACH) {
              mo_add(w1, x[m], -lr1 * d1[m]);
              mo_add(w2, h[m], -lr2 * d2[m]);
              if constexpr (VACC)
                mo_add(v2, -lr2 * dk[m], ho[m]);
              else
                mo_add_v(v2, -lr2 * dk[m], ho[m]);
              ba = fmaf(-lr1, d1[m], ba);
              bb = fmaf(-lr2, d2[m], bb);
            } else {
              mo_add(g1, x[m], d1[m]);
              mo_add(g2, h[m], d2[m]);
              gb1 += d1[m];
              gb2 += d2[m];
            }
          }
        if (EACH && p1.part == 0) {
          b1[o1] = ba;
          b2[o1] = bb;
        }
      }
    }
    PHASE(6);
    // ---------------- updates (Section 3)
    trained_all += (unsigned)nt;
    if constexpr (!EACH) if (nt) {
      c1 += (unsigned)nt;
      c2 += (unsigned)nt;
      c3 += (unsigned)nt;
      auto step = [&](auto& w, auto& g, float f) {
#pragma unroll
        for (int u = 0; u < (int)(sizeof(w) / sizeof(v4f)); ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            w[u][e] = fmaf(f, g[u][e], w[u][e]);
            g[u][e] = 0.f;
          }
      };
      if ((int)c3 >= uni(D->node[2].muf)) {
        const float f = -lr3 * (uni(D->node[2].mean) ? 1.f / (float)c3 : 1.f);
        step(w3, g3, f);
        if (wave == 0) b3[lane] = fmaf(f, gb3, b3[lane]);
        gb3 = 0.f;
        c3 = 0;
        u3++;
        mo_rows_back(T, w3, p3);
        lds_barrier();
        mo_cols(T, v3, q3);
        lds_barrier();
        if (books && tid == 0 && s_log_cap) mo_log(D, 2, 2, 0);
      }
      if ((int)c2 >= uni(D->node[1].muf)) {
        const float f = -lr2 * (uni(D->node[1].mean) ? 1.f / (float)c2 : 1.f);
        step(w2, g2, f);
        if (p1.part == 0) b2[o1] = fmaf(f, gb2, b2[o1]);
        gb2 = 0.f;
        c2 = 0;
        u2++;
        mo_rows_back(T, w2, p2);
        lds_barrier();
        mo_cols(T, v2, p2);
        lds_barrier();
        if (books && tid == 0 && s_log_cap) mo_log(D, 1, 2, 0);
      }
      if ((int)c1 >= uni(D->node[0].muf)) {
        const float f = -lr1 * (uni(D->node[0].mean) ? 1.f / (float)c1 : 1.f);
        step(w1, g1, f);
        if (p1.part == 0) b1[o1] = fmaf(f, gb1, b1[o1]);
        gb1 = 0.f;
        c1 = 0;
        u1++;
        if (books && tid == 0 && s_log_cap) mo_log(D, 0, 2, 0);
      }
    }
    done += (unsigned)n;
    PHASE(7);
  }
  __syncthreads();
  const int tid = threadIdx.x, o1 = p1.out0 + (tid & 63);
  if (tid == 0) {
    D->clock[1] = wall_clock64();
    const unsigned mak = (unsigned)D->mak;
    D->ctl[3] = updates();
    D->ctl[4] = D->admit_bounded ? (unsigned)s_mo_adm.most : mak < n_total ? mak : n_total;
    D->ctl[5] = (unsigned)s_mo_adm.limit;
  }
  if (tid < 3) {   // the layers' records and counters
    const GQ WorkerDev& w = D->worker[1 + tid];
    if (w.log_cap) *w.log_n = s_mo_logn[tid];
    w.stats[1] = done + (tid < 2 ? trained_all : 0u);   // the last layer turns a message round in place
    w.stats[2] = groups;
    w.stats[3] = (unsigned long long)(wall_clock64() - t_begin);
  }
  if (!train) return;
  // ---- parameters, waiting gradients and counters back
  GQ float *const W1 = uni_gq<float>(D->node[0].P), *const W2 = uni_gq<float>(D->node[1].P), *const W3 = uni_gq<float>(D->node[2].P);
  mo_rows_back(T, w2, p2);
  mo_rows_back(T1, w1, p1);   // where the stages' arrays lay
  __syncthreads();
  mo_tile_store(T, W2, H, H);
  mo_tile_store(T1, W1, H, C1);
  __syncthreads();
  mo_rows_back(T, w3, p3);
  __syncthreads();
  mo_tile_store(T, W3, K, H);
  if (tid < H) {
    W1[H * C1 + tid] = b1[tid];
    W2[H * H + tid] = b2[tid];
  }
  if (tid < K) W3[K * H + tid] = b3[tid];
  if constexpr (!EACH) {
    GQ float *const G1 = uni_gq<float>(D->node[0].G), *const G2 = uni_gq<float>(D->node[1].G), *const G3 = uni_gq<float>(D->node[2].G);
    __syncthreads();
    mo_rows_back(T, g2, p2);
    mo_rows_back(T1, g1, p1);
    __syncthreads();
    mo_tile_store(T, G2, H, H);
    mo_tile_store(T1, G1, H, C1);
    __syncthreads();
    mo_rows_back(T, g3, p3);
    __syncthreads();
    mo_tile_store(T, G3, K, H);
    if (tid < K) G3[K * H + tid] = gb3;
    if (p1.part == 0 && o1 < H) {
      G1[H * C1 + o1] = gb1;
      G2[H * H + o1] = gb2;
    }
  }
  if (tid < 3) {
    unsigned* ws = D->worker[1 + tid].wstate;
    ws[0] = tid == 0 ? c1 : tid == 1 ? c2 : c3;
    ws[1] += EACH ? trained_all : tid == 0 ? u1 : tid == 1 ? u2 : u3;
  }
}

// Worker 0 of a replica that mlp_one_fits.
__device__ __forceinline__ void role_mlp_whole(const GQ AmpDev* D, const GQ WorkerDev* W) {
  const bool wide = D->d_in > 64;
  if (D->hidden > 64) {
    if (!mlp_one_each(D))
      role_mlp_one<false, true, 2>(D, W);
    else if (wide)
      role_mlp_one<true, true, 4>(D, W);
    else
      role_mlp_one<true, true, 2>(D, W);
  } else if (mlp_one_each(D)) {
    if (wide)
      role_mlp_one<true, false, 2>(D, W);
    else
      role_mlp_one<true, false, 1>(D, W);
  } else {
    role_mlp_one<false, false, 2>(D, W);
  }
}
