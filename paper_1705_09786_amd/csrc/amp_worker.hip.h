// What every model's persistent kernel shares: the controller (worker 0), the tail of a one-message-at-a-time backward
// step, and the kernel's frame -- which worker a workgroup plays, its utilisation counters and event record.
#pragma once
#include "amp_common.hip.h"

struct Lds {
  float* p;
  __device__ __forceinline__ float* take(int n) {
    float* r = p;
    p += (n + 3) & ~3;
    return r;
  }
};

__shared__ unsigned s_ctl[4];
__shared__ unsigned s_logn;
__shared__ float s_loss;
__shared__ int s_pred;

#define LOG(node, kind, seq, local)                                         \
  do {                                                                      \
    if (threadIdx.x == 0) log_event(D, W, &s_logn, node, kind, seq, local); \
  } while (0)

// ============================================================ controller
// Single-thread wait on the controller's ring.
__device__ __forceinline__ bool ctrl_wait(const GQ AmpDev* D, const GQ RingDev& r, unsigned& head, unsigned& code) {
  const unsigned want = head + 1u;
  GQ unsigned long long* slot = (GQ unsigned long long*)&r.ent[head & r.mask];
  const long long t0 = wall_clock64();
  unsigned spins = 0;
  for (;;) {
    const unsigned long long e = __hip_atomic_load(slot, __ATOMIC_RELAXED, AGENT);
    if ((unsigned)(e >> 32) == want) {   // the controller reads nothing of a payload: no acquire
      code = (unsigned)e;
      head++;
      return true;
    }
    if ((++spins & 7u) == 0u) {
      if (ld_u32(&D->ctl[0])) return false;
      if (wall_clock64() - t0 > D->watchdog_ticks) {
        raise_abort(D, ABORT_WATCHDOG, 0);
        return false;
      }
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

__device__ __noinline__ void role_ctrl(const GQ AmpDev* D, const GQ WorkerDev* W) {
  float* lds = amp_lds;
  if (threadIdx.x == 0) {
    int* freelist = (int*)lds;
    const int mak = D->mak;
    int nfree = mak;
    for (int i = 0; i < mak; ++i) freelist[i] = mak - 1 - i;
    unsigned next = 0, retired = 0, head = 0;
    int active = 0, max_active = 0;
    // Admission.  Greedy: a new instance whenever fewer than max_active_keys are in flight -- at a high
    // max_active_keys the gradients then go stale and training can become unstable (Appendix B, MNIST, which asks
    // for a better schedule).  Staleness-bounded: the number in flight is a limit of its own, between 1 and
    // max_active_keys, which starts at 1, grows by one with every instance that retires having seen at most
    // max_staleness updates per worker during its life, and shrinks by one with every instance that saw more.
    const bool bounded = D->admit_bounded != 0;
    unsigned* upd_at = (unsigned*)(freelist + mak);   // [slot] updates applied so far when the slot's instance was admitted
    int limit = bounded ? 1 : mak;
    const float per_worker = 1.f / (float)(D->n_updaters > 0 ? D->n_updaters : 1);
    const unsigned n_total = D->n_total, n_inst = (unsigned)D->data.n_inst;
    const GQ int* adm = (const GQ int*)D->adm_inst;
    unsigned in_order = 0;   // without an admission list: the data set's instances in order, over and over
    // Synchronisation of a replicated node's copies (Section 5): after every sync_every retirements a request goes to
    // every copy's ring; a new round waits until every copy has reported that it loaded the previous one.
    const int model = D->model;
    const Ring first = ring_regs(D, 1);
    const int NR = model == 2 ? D->node_replicas : 1;
    const unsigned sync_every = NR > 1 ? (unsigned)D->sync_every : 0u;
    unsigned sync_round = 0, sync_due = 0;
    int sync_acks = NR;
    const GQ RingDev& mine = D->ring[W->ring];
    D->clock[0] = wall_clock64();
    bool ok = true;
    while (retired < n_total && ok) {
      while (active < limit && next < n_total) {
        const int s = freelist[--nfree];
        const unsigned seq = s_first_seq + next;
        // which instance this admission is, and whether it only runs forward (training and inference instances
        // share a launch: Section 1)
        const int word = adm ? adm[next] : (int)in_order, inst = word & 0x7fffffff;
        if (++in_order == n_inst) in_order = 0;
        if (bounded) upd_at[s] = ld_u32(&D->ctl[3]);
        D->slot_seq[s] = seq;
        D->slot_inst[s] = word;
        log_event(D, W, &s_logn, 0, 3, seq, word < 0 ? 1u : 0u);
        if (model == 3) {
          // tree: the slot's instance facts for the workers, then one token message per leaf to the lookup (worker 1)
          const int toff = D->data.tok_off[inst], L = D->data.tok_off[inst + 1] - toff;
          int* sm = D->smeta + 4 * s;
          sm[0] = (int)seq;
          sm[1] = L;
          sm[2] = D->data.node_off[inst];
          sm[3] = toff;
          fence_release();
          const unsigned t = ring_reserve(D->ring[1], L);
          for (int l = 0; l < L; ++l) ring_put(D->ring[1], t + l, MSG_MAKE(0, s, l));
        } else {
          if (model == 2) {
            // RNN: admission number, length, instance, token offset
            const int toff = D->data.tok_off[inst];
            int* sm = D->smeta + 4 * s;
            sm[0] = (int)seq;
            sm[1] = D->data.tok_off[inst + 1] - toff;
            sm[2] = inst;
            sm[3] = toff;
          }
          fence_release();
          if (model == 1) {
            // MLP: the message carries the instance; this is the ring's only producer
            ring_put(first, next, MSG_MAKE(0, s, MLP_LOCAL(inst, word < 0)));
          } else {
            // RNN with a replicated cell: the Cond in front of the copies routes on the admission number
            const int rep = model == 2 ? (int)(seq % (unsigned)D->node_replicas) : 0;
            ring_post(D->ring[rep == 0 ? 1 : 2 + rep], MSG_MAKE(0, s, 0));
          }
        }
        next++;
        active++;
        if (active > max_active) max_active = active;
      }
      unsigned code;
      ok = ctrl_wait(D, mine, head, code);
      if (ok && MSG_SLOT(code) == MSG_CTL_SLOT) {
        sync_acks++;   // a copy has loaded the round's mean
      } else if (ok) {
        const int s = MSG_SLOT(code);
        log_event(D, W, &s_logn, 0, 4, D->slot_seq[s], 0);
        freelist[nfree++] = s;
        active--;
        retired++;
        if (bounded) {
          const float seen = (float)(ld_u32(&D->ctl[3]) - upd_at[s]) * per_worker;
          if (seen > D->max_staleness)
            limit = limit > 1 ? limit - 1 : 1;
          else
            limit = limit < mak ? limit + 1 : mak;
        }
        if (sync_every && retired % sync_every == 0u) sync_due++;
      }
      if (sync_due && sync_acks == NR && retired < n_total) {
        sync_due = 0;   // requests that fell due while a round was under way merge into one
        sync_acks = 0;
        sync_round++;
        for (int r = 0; r < NR; ++r) ring_post(D->ring[r == 0 ? 1 : 2 + r], MSG_MAKE(0, MSG_CTL_SLOT, sync_round << 1));
      }
    }
    D->clock[1] = wall_clock64();
    D->ctl[4] = (unsigned)max_active;
    D->ctl[5] = (unsigned)limit;
    fence_release();
    __hip_atomic_store((GQ unsigned*)&D->ctl[1], 1u, __ATOMIC_RELAXED, AGENT);
  }
}

// ============================================================ shared tail of a dense backward
// Counts the gradient, updates when min_update_frequency is reached.
__device__ __forceinline__ void count_and_update(const GQ AmpDev* D, const GQ WorkerDev* W, const GQ NodeDev& nd, const Tile& t,
                                                 float* Wl, float* bl, unsigned& count, unsigned& tstep) {
  count++;
  if ((int)count >= nd.muf) {
    tstep++;
    if (threadIdx.x == 0) note_update(D);
    tile_update(nd, t, Wl, bl, count, tstep);
    count = 0;
    LOG(W->node, 2, 0, 0);
  }
}

// ============================================================ the kernel's frame
// `work(D, W)` runs the role of worker W until the launch is over.  `whole(D)`: worker 0's workgroup does the work of the whole
// replica, by work(D, worker 0), and keeps the other workers' records; theirs leave at once.
template <class Whole, class Work>
__device__ __forceinline__ void persistent_worker(const AmpDev* Dp, int workers_per_replica, int n_replicas, int xcd_packed,
                                                  const AmpLaunch& args, Whole whole, Work work) {
  // Every replica has its own descriptor.  Plain mapping: replica r = blocks [r * workers_per_replica, (r + 1) *
  // workers_per_replica).  Packed mapping: workgroups are dealt to the 8 XCDs in turn, from the XCD on at which the stream's
  // hardware queue starts (another one for every queue that the device has open, of this process or others), so blocks of
  // one index modulo 8 share an XCD; all workers of a replica take blocks of one residue, replicas x, x + 8, ... share an XCD,
  // and a replica's rings, stash and joins stay in one L2.  Blocks without a worker leave at once.
  int replica, wi;
  if (xcd_packed) {
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
    replica = x + 8 * (j / workers_per_replica);
    wi = j % workers_per_replica;
    if (replica >= n_replicas) return;
  } else {
    replica = blockIdx.x / workers_per_replica;
    wi = blockIdx.x - replica * workers_per_replica;
  }
  const GQ AmpDev* D = (const GQ AmpDev*)Dp + replica;
  const GQ WorkerDev* W = &D->worker[wi];
  long long t_begin = 0;
  const int xcc = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & 0xf);   // this workgroup's die: hardware register XCC_ID (id 20), bits 3:0
  const bool alone = whole(D);
  if (alone && wi != 0) {
    if (threadIdx.x == 0) W->stats[12] = (unsigned long long)xcc;
    return;
  }
  if (threadIdx.x == 0) {
    // packed: the whole replica shares one L2 if its workgroups really run on one die; releases then skip the L2 write-back.
    // The first to arrive says which die that is; one that finds itself elsewhere stops the replica before it has exchanged anything.
    s_nowb = 0;
    if (xcd_packed && !alone) {
      unsigned die = 0u;
      const bool first = __hip_atomic_compare_exchange_strong((GQ unsigned*)&D->ctl[7], &die, (unsigned)xcc + 1u, __ATOMIC_RELAXED, __ATOMIC_RELAXED, AGENT);
      s_nowb = first || die == (unsigned)xcc + 1u ? 1 : -1;
    }
    s_logn = 0;
    s_first_seq = args.first_seq[replica];
    s_bounded = D->admit_bounded;
    s_log_cap = W->tile == 0 ? W->log_cap : 0u;
    s_log_ptr = W->log;
    if (W->node >= 0) hold_node_opt(D->node[W->node]);
    for (int i = 0; i < AMP_NSTAT; ++i) s_stat[i] = 0;
    t_begin = wall_clock64();
  }
  __syncthreads();
  if (s_nowb < 0) {
    if (threadIdx.x == 0) {
      raise_abort(D, ABORT_PLACEMENT, wi);
      W->stats[12] = (unsigned long long)xcc;
    }
    return;
  }
  if (W->role == ROLE_CTRL && !alone)
    role_ctrl(D, W);
  else
    work(D, W);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (W->log_cap) *W->log_n = s_logn;
    for (int i = 0; i < AMP_NSTAT; ++i) W->stats[i] = s_stat[i];
    W->stats[3] = (unsigned long long)(wall_clock64() - t_begin);
    W->stats[12] = (unsigned long long)xcc;
  }
}


// Launches one model's persistent kernel.
static inline hipError_t launch_persistent(const void* kernel, bool& attr_set, const AmpDev* devs, int n_replicas,
                                           int workers_per_replica, const AmpLaunch* args, hipStream_t stream) {
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, AMP_DYN_LDS_BYTES);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  // One XCD has 32 CUs: the packed mapping needs the replicas that share an XCD to fit it.  Measured: replicas
  // gain from staying inside one L2 (15 Tree-LSTM replicas 184k -> 256k trees/s), and again from releases without
  // an L2 write-back, which only a packed replica can do (16 replicas 316k -> 409k trees/s).  A single pipeline of up to 12
  // workers is packed too (the RNN with eight copies of its cell, 10 workers, 105k -> 112k sequences/s; the unsplit 10-worker
  // graph pipeline the same either way).  A longer one is spread: packed, it would leave another launch that runs at the same time
  // -- a second context on a stream or in a process of its own -- too few CUs on that die, and two launches that hold a part of one die
  // each would wait for the rest of it until their watchdogs end them.  (What packing gave trees whose cells all keep their
  // inputs on the CU: 2,136 trees on 30 workers 39.75 -> 39.55 ms, evaluation of 1,101 12.4 -> 11.7; 17 graph workers 60.6 spread
  // against 60.7, 16 workers of the older tree cell 69.2 against 70.2.)
  const int per_xcd = (n_replicas + 7) / 8;
  const bool packed = per_xcd * workers_per_replica <= 32 && (n_replicas > 1 || workers_per_replica <= 12);
  const int grid = packed ? 8 * per_xcd * workers_per_replica : n_replicas * workers_per_replica;
  int packed_arg = packed ? 1 : 0;
  AmpLaunch by_value = *args;
  void* params[] = {&devs, &workers_per_replica, &n_replicas, &packed_arg, &by_value};
  return hipLaunchKernel(kernel, dim3(grid), dim3(AMP_THREADS), params, AMP_DYN_LDS_BYTES, stream);
}

// Defines model `name`'s kernel amp_persistent_<name> and its launcher amp_launch_<name>; `whole` says whether worker 0 of a
// replica (D) does all of its work, and the macro's last argument is the statement that runs the role of worker (D, W).
#define AMP_PERSISTENT_KERNEL(name, whole, ...)                                                                                    \
  extern "C" __global__ void __launch_bounds__(AMP_THREADS) amp_persistent_##name(                                          \
      const AmpDev* Dp, int workers_per_replica, int n_replicas, int xcd_packed, AmpLaunch args) {                          \
    persistent_worker(Dp, workers_per_replica, n_replicas, xcd_packed, args, [](const GQ AmpDev* D) { return whole; },      \
                      [](const GQ AmpDev* D, const GQ WorkerDev* W) { __VA_ARGS__ });                                       \
  }                                                                                                                         \
  extern "C" hipError_t amp_launch_##name(const AmpDev* devs, int n_replicas, int workers_per_replica, const AmpLaunch* a,  \
                                          hipStream_t stream) {                                                             \
    static bool attr_set = false;                                                                                           \
    return launch_persistent((const void*)amp_persistent_##name, attr_set, devs, n_replicas, workers_per_replica, a, stream); \
  }
