// Persistent AMP training kernel for gfx950.
//
// One launch = one amp_train / amp_eval call.  Workgroup w plays worker w
// (Appendix A of the paper: a worker hosts one or more IR nodes and is fed by
// a multi-producer queue): it keeps its nodes' weights in LDS, takes keyed
// messages from its ring, runs the node's forward or backward transform,
// accumulates the gradient, applies the node's own update once
// min_update_frequency gradients have arrived (Section 3), and posts the
// resulting messages.  Worker 0 is the controller (Section 4): it admits
// instances while fewer than max_active_keys are active and retires them when
// their last backward message has come back.
//
// Control-flow nodes of the IR (Cond, Phi, Isu, Concat, Bcast, Group,
// Ungroup, Flatmap) are pure functions of the message state; here they are
// the index arithmetic a producer performs when it decides where a result
// goes, plus arrival counters where several messages must meet.
#include <hip/hip_runtime.h>
#include <mutex>
#include "amp_common.hip.h"

// One kernel per model, each in a source file of its own (amp_mlp.hip, amp_rnn.hip, amp_tree.hip, amp_ggnn.hip).
#define AMP_LAUNCHER(name) \
  extern "C" hipError_t amp_launch_##name(const AmpDev*, int, int, const AmpLaunch*, hipStream_t)
AMP_LAUNCHER(mlp);
AMP_LAUNCHER(rnn);
AMP_LAUNCHER(tree);
AMP_LAUNCHER(ggnn);

extern "C" hipError_t amp_launch(int model, const AmpDev* devs, int n_replicas, int workers_per_replica, const AmpLaunch* args,
                                 hipStream_t stream) {
  switch (model) {
    case 1: return amp_launch_mlp(devs, n_replicas, workers_per_replica, args, stream);
    case 2: return amp_launch_rnn(devs, n_replicas, workers_per_replica, args, stream);
    case 3: return amp_launch_tree(devs, n_replicas, workers_per_replica, args, stream);
    case 4: return amp_launch_ggnn(devs, n_replicas, workers_per_replica, args, stream);
    default: return hipErrorInvalidValue;
  }
}

// ============================================================ around a launch
// Clears a contiguous range and b_count equally spaced ones: one launch for everything that must be zero before a
// launch (24 replicas took 24 memsets of about 3 us each).  Ranges are whole 16-byte groups.
__global__ void __launch_bounds__(256) amp_clear_kernel(v4i* a, size_t a16, v4i* b, size_t b16, size_t b_stride16, size_t total) {
  const v4i zero = {0, 0, 0, 0};
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    if (i < a16) {
      a[i] = zero;
    } else {
      const size_t j = i - a16, r = j / b16;
      b[r * b_stride16 + (j - r * b16)] = zero;
    }
  }
}

extern "C" hipError_t amp_clear(void* a, size_t a_bytes, void* b, size_t b_bytes, size_t b_stride, int b_count, hipStream_t stream) {
  const size_t a16 = a_bytes / 16, b16 = b_bytes / 16, total = a16 + b16 * (size_t)b_count;
  if (total == 0) return hipSuccess;
  const size_t blocks = (total + 255) / 256;
  hipLaunchKernelGGL(amp_clear_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, stream, (v4i*)a, a16, (v4i*)b, b16,
                     b_stride / 16, total);
  return hipGetLastError();
}

// End-of-epoch synchronisation of replicas (Section 5): every replica's copy of the parameters becomes the mean over
// the replicas, summed in replica order.  Bound by HBM traffic (every copy is read and written once): 16-byte
// accesses, eight replicas' values in flight.
__global__ void __launch_bounds__(256) amp_average_kernel(v4f* p0, size_t stride4, int n_replicas, size_t n4) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n4) return;
  v4f s = {0.f, 0.f, 0.f, 0.f};
  for (int r0 = 0; r0 < n_replicas; r0 += 8) {
    v4f v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = p0[(size_t)(r0 + k < n_replicas ? r0 + k : n_replicas - 1) * stride4 + i];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (r0 + k < n_replicas) s += v[k];
  }
  const float n = (float)n_replicas;
  s = (v4f){s.x / n, s.y / n, s.z / n, s.w / n};
  for (int r = 0; r < n_replicas; ++r) p0[(size_t)r * stride4 + i] = s;
}

// n and the stride in floats; copies start 16-byte aligned and are padded to a multiple of 16 bytes.
extern "C" hipError_t amp_average(float* p0, size_t stride_floats, int n_replicas, size_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const size_t n4 = (n + 3) / 4;
  hipLaunchKernelGGL(amp_average_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, stream, (v4f*)p0, stride_floats / 4,
                     n_replicas, n4);
  return hipGetLastError();
}

// ============================================================ built-in arena
// Device memory that exists without any allocation call: amp_create_static hands it to a context in place of a
// caller-provided arena.  Every GPU the library's code object is loaded on holds its own copy, at its own address,
// until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the address it
// returns (looked up once per device, with that device current) is what kernels, copies and clears are given.
static __device__ __align__(256) unsigned char scratch[AMP_STATIC_ARENA_BYTES];

extern "C" hipError_t amp_static_arena(void** ptr, size_t* bytes) {
  constexpr int MAX_DEV = 64;
  static std::mutex mu;
  static void* addr[MAX_DEV] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEV) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p || ((uintptr_t)p & 255)) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  *bytes = AMP_STATIC_ARENA_BYTES;
  return hipSuccess;
}

// ============================================================ peak micro-benchmarks
// What the roofline fractions are measured against can itself be measured: the
// LDS read rate of one workgroup per CU shaped like a worker (512 threads,
// 16-byte reads, several independent reads in flight), and the HBM read rate
// of a grid-wide streaming sum.
extern "C" __global__ void __launch_bounds__(AMP_THREADS) amp_peak_lds_kernel(int iters, float* sink) {
  LDSQ float* l = (LDSQ float*)amp_lds;
  const int nfl = AMP_DYN_LDS_BYTES / 4;
  for (int i = threadIdx.x; i < nfl; i += AMP_THREADS) l[i] = (float)(i & 7);
  __syncthreads();
  // each thread walks the whole LDS in 16-byte steps, eight reads per round
  const int nv = nfl / 4;   // 16-byte groups
  v4f a[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) a[k] = (v4f){0.f, 0.f, 0.f, 0.f};
  int pos = threadIdx.x;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      a[k] += *(const LDSQ v4f*)(l + 4 * pos);
      pos += AMP_THREADS;
      if (pos >= nv) pos -= nv;
    }
  }
  v4f r = a[0];
#pragma unroll
  for (int k = 1; k < 8; ++k) r += a[k];
  if (r.x + r.y + r.z + r.w == -1.f) sink[0] = r.x;   // never true: keeps the reads alive
}

extern "C" __global__ void __launch_bounds__(256) amp_peak_hbm_kernel(const v4f* src, size_t n16, float* sink) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  v4f a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0, a2 = a0, a3 = a0;
  for (; i + 3 * stride < n16; i += 4 * stride) {
    a0 += src[i];
    a1 += src[i + stride];
    a2 += src[i + 2 * stride];
    a3 += src[i + 3 * stride];
  }
  for (; i < n16; i += stride) a0 += src[i];
  const v4f r = a0 + a1 + a2 + a3;
  if (r.x + r.y + r.z + r.w == -1.2345f) sink[0] = r.x;
}

// Launches the LDS benchmark on n_wg workgroups (one per CU: the dynamic LDS
// size allows no second one) and returns the seconds the timed launch took
// and the bytes it read per workgroup.
extern "C" hipError_t amp_peak_lds_launch(int n_wg, int iters, float* sink, hipStream_t stream, double* seconds,
                                          double* bytes_per_wg) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)amp_peak_lds_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       AMP_DYN_LDS_BYTES);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipEvent_t t0, t1;
  hipError_t e;
  if ((e = hipEventCreate(&t0)) != hipSuccess) return e;
  if ((e = hipEventCreate(&t1)) != hipSuccess) return e;
  hipLaunchKernelGGL(amp_peak_lds_kernel, dim3(n_wg), dim3(AMP_THREADS), AMP_DYN_LDS_BYTES, stream, iters / 8 + 1, sink);   // warm-up
  (void)hipEventRecord(t0, stream);
  hipLaunchKernelGGL(amp_peak_lds_kernel, dim3(n_wg), dim3(AMP_THREADS), AMP_DYN_LDS_BYTES, stream, iters, sink);
  (void)hipEventRecord(t1, stream);
  if ((e = hipEventSynchronize(t1)) != hipSuccess) return e;
  float ms = 0.f;
  (void)hipEventElapsedTime(&ms, t0, t1);
  (void)hipEventDestroy(t0);
  (void)hipEventDestroy(t1);
  *seconds = ms * 1e-3;
  *bytes_per_wg = (double)iters * 8.0 * AMP_THREADS * 16.0;
  return hipGetLastError();
}

extern "C" hipError_t amp_peak_hbm_launch(const void* src, size_t bytes, float* sink, hipStream_t stream, double* seconds) {
  hipEvent_t t0, t1;
  hipError_t e;
  if ((e = hipEventCreate(&t0)) != hipSuccess) return e;
  if ((e = hipEventCreate(&t1)) != hipSuccess) return e;
  const size_t n16 = bytes / 16;
  const int grid = 256 * 16;
  hipLaunchKernelGGL(amp_peak_hbm_kernel, dim3(grid), dim3(256), 0, stream, (const v4f*)src, n16, sink);   // warm-up
  (void)hipEventRecord(t0, stream);
  hipLaunchKernelGGL(amp_peak_hbm_kernel, dim3(grid), dim3(256), 0, stream, (const v4f*)src, n16, sink);
  (void)hipEventRecord(t1, stream);
  if ((e = hipEventSynchronize(t1)) != hipSuccess) return e;
  float ms = 0.f;
  (void)hipEventElapsedTime(&ms, t0, t1);
  (void)hipEventDestroy(t0);
  (void)hipEventDestroy(t1);
  *seconds = ms * 1e-3;
  return hipGetLastError();
}
