// ntc_cluster.hip -- Stage 2 of the paper's texture pipeline (Alg. "Overall
// texture processing pipeline"): k-means clustering of one feature vector per
// texture into m groups; the group labels are the texture -> decoder map c(i)
// that the decode path reads.  The paper clusters CLIP embeddings (Stage 1);
// any per-texture features can be given.
//
// Lloyd's algorithm in fp64, for up to max_iter iterations without host
// synchronisation.  Three pieces of device code:
//   seed   : centroid j = features of texture init[j]; flags cleared.
//   assign : one wave per texture; squared Euclidean distance to kAssignCols
//            centroids at a time (lanes stride the dimensions, butterfly sums),
//            nearest centroid with ties to the lower index.
//   update : one wave per (cluster, 64 dimensions); the wave lists the cluster's
//            members in ascending order (ballots over the labels), then every
//            lane sums its dimension over the list and divides by the count; an
//            empty cluster keeps its centroid.  Sizes k_g go to counts[j].
//
// Where the work of an iteration is small (kPersistWork), one launch runs every
// iteration on at most one workgroup per CU, with a grid-wide wait after the
// assignment and after the update, and stops when no label changes; two launches
// an iteration cost 3.4 us each on the queue, also after convergence (100
// iterations of 512 textures x 512 dimensions into 16 groups: 690 of 715 us).
// Every wait is bounded: a workgroup whose wait runs out returns, and the
// kernel behind, one workgroup, runs the clustering again from the seeds when
// the flags say that the first did not finish (its grid was not resident at
// once, which another stream's long kernels can cause).  Same sums in the same
// order on every path, so the results are the same bits.  Larger problems take
// an assignment and an update launch per iteration, and a per-iteration flag
// lets every launch after convergence return at once.
//
// What bounds it: latency.  Per iteration of 512 x 512 into 16 groups the
// assignment takes 8-10 us (two rounds of loads per 8 centroids), each wait
// 3.5 us (the L2s are written back and invalidated) and the update 6-9 us (the
// member rows of the largest cluster, added in order); 3 iterations and the
// launches: 683 us before, 105 us now.  20,000 x 512 into 300 groups, 4
// iterations on the launch-per-iteration path: 17.3 -> 7.0 ms.
#include "ntc_internal.h"

namespace ntc {
namespace {

// n * m * dim up to here: one persistent launch (at 2^28 an iteration's
// arithmetic is about 50 us on the whole chip, against 7 us for two launches).
constexpr int64_t kPersistWork = (int64_t)1 << 28;
constexpr int64_t kPersistPoints = 65536;  // update: every unit scans all labels
constexpr int kPersistGroups = 256;        // workgroups, at most (fields below hold 1023)
constexpr uint64_t kWaitTicks = 2000000;   // 20 ms of the 100 MHz counter
constexpr int kAssignCols = 8;             // centroids a wave compares at once
constexpr int kListRows = 16;              // update: labels a wave lists at once, in rows of 64
constexpr int kListLen = kListRows * kWave;
constexpr int kSumBatch = 32;              // update: member rows in flight

// Seeds passed by value (m <= kArgSeeds): no copy to wait for.
constexpr int kArgSeeds = 256;
struct Seeds {
  uint32_t v[kArgSeeds];
};

// flags[t] of iteration t: bits 0-9 workgroups past the assignment, bits 10-19
// those that changed a label, bits 20-29 those past the update.  The
// launch-per-iteration path and the one-workgroup kernel only set kChanged.
constexpr uint32_t kField = 1023u;
constexpr uint32_t kAssigned = 1u, kChanged = 1u << 10, kUpdated = 1u << 20;
__host__ __device__ inline bool any_change(uint32_t flag) { return ((flag >> 10) & kField) != 0; }

struct Problem {
  const float *features;
  int32_t n, dim, m;
  double *centroids;
  uint32_t *assign, *counts, *flags;
  int32_t max_iter;
};

// seeds NULL: they come by value.
__device__ __forceinline__ void seed_centroids(const Problem &p, const Seeds &arg,
                                               const uint32_t *seeds, uint32_t j) {
  const uint32_t row = seeds ? seeds[j] : arg.v[j];
  const float *x = p.features + (size_t)row * p.dim;
  for (int k = threadIdx.x; k < p.dim; k += blockDim.x)
    p.centroids[(size_t)j * p.dim + k] = (double)x[k];
}

__global__ void __launch_bounds__(kBlock)
kmeans_seed(const Problem p, const Seeds arg, const uint32_t *__restrict__ seeds) {
  seed_centroids(p, arg, seeds, blockIdx.x);
  if (blockIdx.x == 0)
    for (int t = threadIdx.x; t < p.max_iter; t += kBlock) p.flags[t] = 0;
}

// Butterfly sums of kAssignCols values over the wave: the first three steps
// halve the values a lane carries, so lane l ends with the total of value
// bitrev3(l & 7); each total is the sum a full butterfly gives, bit for bit
// (the same pairs are added at every step).
__device__ __forceinline__ double wave_sum8(double (&v)[kAssignCols], uint32_t lane) {
  static_assert(kAssignCols == 8, "three halving steps");
#pragma unroll
  for (int step = 0; step < 3; ++step) {
    const int half = 4 >> step, s = 1 << step;
    const bool up = (lane >> step) & 1;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const double keep = up ? v[half + i] : v[i], give = up ? v[i] : v[half + i];
      v[i] = keep + __shfl_xor(give, s, kWave);
    }
  }
#pragma unroll
  for (int s = 8; s < kWave; s <<= 1) v[0] += __shfl_xor(v[0], s, kWave);
  return v[0];
}

// Labels of textures wave, wave + n_waves, ...; returns whether this lane's wave
// changed one (every label counts as changed at t = 0).  DEPTH: steps of 64
// dimensions in flight.  One texture a wave leaves a few waves a CU, so an
// iteration is the latency of its rounds of loads: 512 dimensions in rounds of 2
// steps took 20 us, of 4 steps 9.7 us.
template <int DEPTH>
__device__ __forceinline__ bool assign_rows(const Problem &p, uint32_t wave, uint32_t n_waves,
                                              int32_t t) {
  const uint32_t lane = lane_id();
  const uint32_t col = ((lane & 1) << 2) | (lane & 2) | ((lane >> 2) & 1);  // bitrev3
  bool changed = false;
  for (uint32_t i = wave; i < (uint32_t)p.n; i += n_waves) {
    const float *x = p.features + (size_t)i * p.dim;
    double best = __builtin_inf();
    uint32_t bj = 0;
    for (int32_t j0 = 0; j0 < p.m; j0 += kAssignCols) {
      double s[kAssignCols] = {};
      const double *c[kAssignCols];
#pragma unroll
      for (int q = 0; q < kAssignCols; ++q)  // columns past m repeat the last centroid
        c[q] = p.centroids + (size_t)min(j0 + q, p.m - 1) * p.dim;
      // a lane past the last dimension reads it again and adds nothing
      for (int k0 = 0; k0 < p.dim; k0 += DEPTH * kWave) {
        float xv[DEPTH];
        double cv[DEPTH][kAssignCols];
#pragma unroll
        for (int e = 0; e < DEPTH; ++e) {
          const int k = min(k0 + e * kWave + (int)lane, p.dim - 1);
          xv[e] = x[k];
#pragma unroll
          for (int q = 0; q < kAssignCols; ++q) cv[e][q] = c[q][k];
        }
#pragma unroll
        for (int e = 0; e < DEPTH; ++e) {
          const bool in = k0 + e * kWave + (int)lane < p.dim;
#pragma unroll
          for (int q = 0; q < kAssignCols; ++q) {
            const double d = (double)xv[e] - cv[e][q];
            s[q] = in ? __builtin_fma(d, d, s[q]) : s[q];
          }
        }
      }
      const double total = wave_sum8(s, lane);
      const uint32_t j = (uint32_t)j0 + col;
      if (j < (uint32_t)p.m && total < best) {
        best = total;
        bj = j;
      }
    }
    // the eight lanes of a group hold the candidates: the nearest, ties to the
    // lower index
#pragma unroll
    for (int s = 1; s < kAssignCols; s <<= 1) {
      const double ob = __shfl_xor(best, s, kWave);
      const uint32_t oj = __shfl_xor(bj, s, kWave);
      if (ob < best || (ob == best && oj < bj)) {
        best = ob;
        bj = oj;
      }
    }
    if (lane == 0) {
      changed = changed || t == 0 || p.assign[i] != bj;
      p.assign[i] = bj;
    }
  }
  return changed;
}

__device__ __forceinline__ bool assign_points(const Problem &p, uint32_t wave, uint32_t n_waves,
                                              int32_t t) {
  if (p.dim <= kWave) return assign_rows<1>(p, wave, n_waves, t);
  if (p.dim <= 2 * kWave) return assign_rows<2>(p, wave, n_waves, t);
  if (p.dim <= 4 * kWave) return assign_rows<4>(p, wave, n_waves, t);
  return assign_rows<8>(p, wave, n_waves, t);
}

// Units unit, unit + n_units, ... of the update: unit j * slices + k covers
// dimensions 64 k .. of cluster j.  list: kListLen entries of the wave's own.
__device__ __forceinline__ void update_centroids(const Problem &p, uint32_t wave, uint32_t n_waves,
                                                 uint16_t *list) {
  const uint32_t lane = lane_id();
  const uint32_t slices = ((uint32_t)p.dim + kWave - 1) / kWave;
  const uint64_t units = (uint64_t)p.m * slices;
  for (uint64_t u = wave; u < units; u += n_waves) {
    const uint32_t j = (uint32_t)(u / slices), k = (uint32_t)(u % slices) * kWave + lane;
    const uint32_t kc = k < (uint32_t)p.dim ? k : (uint32_t)p.dim - 1;
    double s = 0.0;
    uint32_t count = 0;
    for (uint32_t base = 0; base < (uint32_t)p.n; base += kListLen) {
      uint32_t lab[kListRows];
#pragma unroll
      for (int r = 0; r < kListRows; ++r) {
        const uint32_t i = base + (uint32_t)r * kWave + lane;
        lab[r] = p.assign[i < (uint32_t)p.n ? i : (uint32_t)p.n - 1];
      }
      uint32_t len = 0;
      __builtin_amdgcn_wave_barrier();  // the previous list has been read
#pragma unroll
      for (int r = 0; r < kListRows; ++r) {
        const uint32_t o = (uint32_t)r * kWave + lane;
        const uint64_t mine = ballot(base + o < (uint32_t)p.n && lab[r] == j);
        if ((mine >> lane) & 1) list[len + lanes_below(mine)] = (uint16_t)o;
        len += (uint32_t)__builtin_popcountll(mine);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const float *rows = p.features + (size_t)base * p.dim + kc;
      for (uint32_t q = 0; q < len; q += kSumBatch) {
        float v[kSumBatch];
#pragma unroll
        for (int e = 0; e < kSumBatch; ++e)
          v[e] = rows[(size_t)list[q + e < len ? q + e : len - 1] * p.dim];
#pragma unroll
        for (int e = 0; e < kSumBatch; ++e)
          if (q + e < len) s += (double)v[e];
      }
      count += len;
    }
    if (count && k < (uint32_t)p.dim) p.centroids[(size_t)j * p.dim + k] = s / (double)count;
    if (k == 0) p.counts[j] = count;
  }
}

__global__ void __launch_bounds__(kBlock) kmeans_assign(const Problem p, int32_t t) {
  if (t > 0 && !any_change(p.flags[t - 1])) return;  // converged at an earlier iteration
  const uint32_t wave = blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
  if (assign_points(p, wave, gridDim.x * kWavesPerBlock, t)) p.flags[t] = kChanged;
}

__global__ void __launch_bounds__(kBlock) kmeans_update(const Problem p, int32_t t) {
  __shared__ uint16_t lists[kWavesPerBlock][kListLen];
  if (!any_change(p.flags[t])) return;  // no label changed: the centroids stand
  const uint32_t w = threadIdx.x / kWave;
  update_centroids(p, blockIdx.x * kWavesPerBlock + w, gridDim.x * kWavesPerBlock, lists[w]);
}

// Adds `add` to *word for this workgroup and waits until the field at `shift`
// holds gridDim.x, at most kWaitTicks; returns the word, or kTimedOut.  What
// every workgroup wrote before its own call is visible after it.
constexpr uint32_t kTimedOut = 0xFFFFFFFFu;
__device__ uint32_t grid_wait(uint32_t *word, uint32_t add, int shift, uint32_t *shared) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    uint32_t v = __hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    bool in = ((v >> shift) & kField) == gridDim.x;
    while (!in && __builtin_amdgcn_s_memrealtime() - t0 < kWaitTicks) {
      __builtin_amdgcn_s_sleep(1);
      v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      in = ((v >> shift) & kField) == gridDim.x;
    }
    __threadfence();
    *shared = in ? v : kTimedOut;
  }
  __syncthreads();
  return *shared;
}

__global__ void __launch_bounds__(kBlock) kmeans_persistent(const Problem p) {
  __shared__ uint16_t lists[kWavesPerBlock][kListLen];
  __shared__ uint32_t word[2];
  const uint32_t w = threadIdx.x / kWave;
  const uint32_t wave = blockIdx.x * kWavesPerBlock + w, n_waves = gridDim.x * kWavesPerBlock;
  for (int32_t t = 0; t < p.max_iter; ++t) {
    const bool changed = __syncthreads_or(assign_points(p, wave, n_waves, t));
    const uint32_t v = grid_wait(p.flags + t, kAssigned + (changed ? kChanged : 0u), 0, &word[0]);
    if (v == kTimedOut || !any_change(v)) return;
    update_centroids(p, wave, n_waves, lists[w]);
    if (grid_wait(p.flags + t, kUpdated, 20, &word[1]) == kTimedOut) return;
  }
}

// One workgroup: returns at once when kmeans_persistent (of `groups` workgroups)
// ran to its end, else runs the clustering from the seeds.
constexpr int kFinishThreads = kBlock;
__global__ void __launch_bounds__(kFinishThreads)
kmeans_finish(const Problem p, const Seeds arg, uint32_t groups) {
  constexpr int kWaves = kFinishThreads / kWave;
  __shared__ uint16_t lists[kWaves][kListLen];
  __shared__ int32_t stop;
  // first iteration after which the grid did not go on
  if (threadIdx.x == 0) stop = p.max_iter;
  __syncthreads();
  for (int32_t t = threadIdx.x; t < p.max_iter; t += kFinishThreads) {
    const uint32_t v = p.flags[t];
    if ((v & kField) != groups || !any_change(v) || ((v >> 20) & kField) != groups)
      atomicMin(&stop, t);
  }
  __syncthreads();
  if (stop == p.max_iter) return;
  const uint32_t at = p.flags[stop];
  if ((at & kField) == groups && !any_change(at)) return;  // converged there
  __syncthreads();
  for (int32_t t = threadIdx.x; t < p.max_iter; t += kFinishThreads) p.flags[t] = 0;
  for (int32_t j = 0; j < p.m; ++j) seed_centroids(p, arg, nullptr, (uint32_t)j);
  const uint32_t w = threadIdx.x / kWave;
  for (int32_t t = 0; t < p.max_iter; ++t) {
    __syncthreads();
    const bool changed = __syncthreads_or(assign_points(p, w, kWaves, t));
    if (!changed) return;
    if (threadIdx.x == 0) p.flags[t] = kChanged;
    update_centroids(p, w, kWaves, lists[w]);
  }
}

}  // namespace

size_t kmeans_workspace_bytes(int32_t m, int32_t max_iter) {
  return ((size_t)m + (size_t)max_iter) * sizeof(uint32_t);
}

int launch_kmeans(const float *features, int32_t n, int32_t dim, int32_t m, const uint32_t *init,
                  int32_t max_iter, uint32_t *assign, double *centroids, uint32_t *counts,
                  void *workspace, hipStream_t stream) {
  uint32_t *dinit = (uint32_t *)workspace;  // [m] seed textures, then [max_iter] flags
  const Problem p = {features, n, dim, m, centroids, assign, counts, dinit + m, max_iter};
  // the seed list is the caller's host memory: by value where it fits a kernel's
  // arguments, else copied before this call returns
  Seeds arg = {};
  const bool by_value = m <= kArgSeeds;
  if (by_value) {
    for (int32_t j = 0; j < m; ++j) arg.v[j] = init[j];
  } else if (hipMemcpyAsync(dinit, init, (size_t)m * sizeof(uint32_t), hipMemcpyHostToDevice,
                            stream) != hipSuccess ||
             hipStreamSynchronize(stream) != hipSuccess) {
    return NTC_ERR_HIP;
  }
  hipLaunchKernelGGL(kmeans_seed, dim3((unsigned)m), dim3(kBlock), 0, stream, p, arg,
                     by_value ? nullptr : dinit);
  const int64_t units = (int64_t)m * ((dim + kWave - 1) / kWave);
  const auto groups_of = [](int64_t waves) { return (waves + kWavesPerBlock - 1) / kWavesPerBlock; };
  if (by_value && n <= kPersistPoints && (int64_t)n * m <= kPersistWork / dim) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return NTC_ERR_HIP;
    int64_t groups = groups_of(n > units ? n : units);
    const int64_t most = cus < kPersistGroups ? cus : kPersistGroups;
    if (groups > most) groups = most;
    hipLaunchKernelGGL(kmeans_persistent, dim3((unsigned)groups), dim3(kBlock), 0, stream, p);
    hipLaunchKernelGGL(kmeans_finish, dim3(1), dim3(kFinishThreads), 0, stream, p, arg,
                       (uint32_t)groups);
    return hip_status(hipGetLastError());
  }
  const int64_t most_units = (int64_t)1 << 20;  // grid stride beyond
  const unsigned assign_blocks = (unsigned)groups_of(n);
  const unsigned update_blocks = (unsigned)groups_of(units < most_units ? units : most_units);
  for (int32_t t = 0; t < max_iter; ++t) {
    hipLaunchKernelGGL(kmeans_assign, dim3(assign_blocks), dim3(kBlock), 0, stream, p, t);
    hipLaunchKernelGGL(kmeans_update, dim3(update_blocks), dim3(kBlock), 0, stream, p, t);
  }
  return hip_status(hipGetLastError());
}

int read_kmeans_state(const void *workspace, int32_t m, int32_t max_iter, int32_t *iterations,
                      int32_t *converged, hipStream_t stream) {
  const uint32_t *flags = (const uint32_t *)workspace + m;
  uint32_t buf[64];
  int32_t done = max_iter, conv = 0;
  for (int32_t t0 = 0; t0 < max_iter && !conv; t0 += 64) {
    const int32_t len = max_iter - t0 < 64 ? max_iter - t0 : 64;
    hipError_t e = hipMemcpyAsync(buf, flags + t0, (size_t)len * sizeof(uint32_t),
                                  hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return NTC_ERR_HIP;
    for (int32_t k = 0; k < len; ++k) {
      if (!any_change(buf[k])) {
        done = t0 + k + 1;
        conv = 1;
        break;
      }
    }
  }
  if (iterations) *iterations = done;
  if (converged) *converged = conv;
  return NTC_OK;
}

}  // namespace ntc
