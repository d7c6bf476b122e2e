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
// iteration on at most one workgroup per CU and stops when no label changes; two
// launches an iteration cost 3.4 us each on the queue, also after convergence
// (100 iterations of 512 textures x 512 dimensions into 16 groups: 690 of 715 us).
// A unit of its work is a share of an iteration's assignment or update.  When all
// its workgroups have started (they count themselves first), each keeps its own
// units through all iterations: static units find their textures in the L2 again.
// When some have not started within kStartTicks (another stream's long kernels can
// hold them back), the units are claimed one by one instead, and nobody waits but
// for units whose workgroups are running, so the launch ends however few of its
// workgroups the device runs at once, and those that start late help with what is
// left.  Same sums in the same order whoever computes a unit, so the results are
// the same bits.  Larger problems take an assignment and an update launch per
// iteration, and a per-iteration flag lets every launch after convergence return at
// once.
//
// What bounds it: latency.  Per iteration of 512 x 512 into 16 groups the
// assignment takes 8-10 us (two rounds of loads per 8 centroids), each wait
// 3.5 us (the L2s are written back and invalidated) and the update 6-9 us (the
// member rows of the largest cluster, added in order); 3 iterations and the
// launches: 690 us with two launches an iteration, 124 now (129 when a kernel
// behind the launch checked whether it had run to its end).  20,000 x 512 into 300 groups, 4
// iterations on the launch-per-iteration path: 17.3 -> 7.0 ms.
#include "ntc_internal.h"

namespace ntc {
namespace {

// n * m * dim up to here: one persistent launch (at 2^28 an iteration's
// arithmetic is about 50 us on the whole chip, against 7 us for two launches).
constexpr int64_t kPersistWork = (int64_t)1 << 28;
constexpr int64_t kPersistPoints = 65536;  // update: every unit scans all labels
constexpr int kPersistGroups = 256;        // units and workgroups, at most (fields below)
constexpr uint64_t kStartTicks = 10000;    // 100 us of the 100 MHz counter
constexpr int kAssignCols = 8;             // centroids a wave compares at once
constexpr int kListRows = 16;              // update: labels a wave lists at once, in rows of 64
constexpr int kListLen = kListRows * kWave;
constexpr int kSumBatch = 32;              // update: member rows in flight

// Seeds passed by value (m <= kArgSeeds): no copy to wait for.
constexpr int kArgSeeds = 256;
struct Seeds {
  uint32_t v[kArgSeeds];
};

// flags[t] of iteration t.  The persistent launch: bits 0-9 claims (the units of
// the assignment, then those of the update, then one past them from each
// workgroup: at most 3 * kPersistGroups), bits 10-18 units assigned, bits 19-27
// those of them that changed a label.  The launches per iteration set kChanged.
constexpr uint32_t kClaim = 1u, kClaims = 1023u, kUnits = 511u;
constexpr uint32_t kAssigned = 1u << 10, kChanged = 1u << 19;
static_assert(3 * kPersistGroups <= kClaims && kPersistGroups <= kUnits, "fields of a flag word");
__host__ __device__ inline bool any_change(uint32_t flag) { return (flag / kChanged & kUnits) != 0; }

// The persistent launch's progress word: bits 0-20 units updated in all iterations,
// bits 21-29 workgroups started, bit 31 units are claimed.
constexpr uint32_t kUpdated = (1u << 21) - 1, kStarted = 1u << 21, kClaiming = 1u << 31;
static_assert((int64_t)kPersistGroups * NTC_KMEANS_MAX_ITER <= kUpdated, "updates of a whole run");
__host__ __device__ inline uint32_t started(uint32_t progress) { return progress / kStarted & kUnits; }

struct Problem {
  const float *features;
  int32_t n, dim, m;
  double *centroids;
  uint32_t *assign, *counts, *flags;
  uint32_t *progress;  // of the persistent launch
  int32_t max_iter;
};

// seeds NULL: they come by value.
__global__ void __launch_bounds__(kBlock)
kmeans_seed(const Problem p, const Seeds arg, const uint32_t *__restrict__ seeds) {
  const uint32_t j = blockIdx.x, row = seeds ? seeds[j] : arg.v[j];
  const float *x = p.features + (size_t)row * p.dim;
  for (int k = threadIdx.x; k < p.dim; k += kBlock)
    p.centroids[(size_t)j * p.dim + k] = (double)x[k];
  if (j == 0) {
    for (int t = threadIdx.x; t < p.max_iter; t += kBlock) p.flags[t] = 0;
    if (!seeds && threadIdx.x == 0) *p.progress = 0;
  }
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

// Adds to a word that workgroups share; returns its old value.
__device__ __forceinline__ uint32_t add_shared(uint32_t *word, uint32_t v) {
  return __hip_atomic_fetch_add(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t read_shared(const uint32_t *word) {
  return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until done(*word), starting from a value `v` that thread 0 has seen;
// returns the word.  What was written before the marks in it is visible after.
template <typename Done>
__device__ __forceinline__ uint32_t wait_until(const uint32_t *word, uint32_t v, Done done,
                                               uint32_t *said) {
  __syncthreads();  // *said has been read
  if (threadIdx.x == 0) {
    while (!done(v)) {
      __builtin_amdgcn_s_sleep(1);
      v = read_shared(word);
    }
    __threadfence();
    *said = v;
  }
  __syncthreads();
  return *said;
}

// Counts this workgroup as started and waits until all `expected` have, or until
// the time is up; returns whether units are claimed.  Every workgroup returns the
// same: kClaiming is only ever set while some have not started.
__device__ __forceinline__ bool start(uint32_t *progress, uint32_t expected, uint32_t *said) {
  if (threadIdx.x == 0) {
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    uint32_t v = add_shared(progress, kStarted) + kStarted;
    while (!(v & kClaiming) && started(v) != expected) {
      if (__builtin_amdgcn_s_memrealtime() - t0 >= kStartTicks) {
        const uint32_t old = atomicCAS(progress, v, v | kClaiming);
        v = old == v ? v | kClaiming : old;
      } else {
        __builtin_amdgcn_s_sleep(1);
        v = read_shared(progress);
      }
    }
    *said = v & kClaiming;
  }
  __syncthreads();
  return *said != 0;
}

// expected: workgroups of the launch.  Every wait ends.  Without claims all
// workgroups are running and each marks its units of a phase before it waits for
// the others'.  With claims a workgroup waits for the assignment of t only once its
// claim in t lies past it, and for the update of t - 1 only once it has left t - 1,
// with a claim past that: all units waited for are claimed, and their workgroups run
// and wait, if at all, for an earlier phase.
__global__ void __launch_bounds__(kBlock)
kmeans_persistent(const Problem p, uint32_t a_units, uint32_t u_units, uint32_t expected) {
  __shared__ uint16_t lists[kWavesPerBlock][kListLen];
  __shared__ uint32_t said[3];
  const uint32_t w = threadIdx.x / kWave;
  const bool claims = start(p.progress, expected, &said[2]);
  uint32_t progress = 0;  // thread 0: as last seen
  for (int32_t t = 0; t < p.max_iter; ++t) {
    uint32_t *word = p.flags + t, seen = 0, unit = blockIdx.x;
    if (claims) {
      if (threadIdx.x == 0) said[0] = add_shared(word, kClaim) & kClaims;
      __syncthreads();
      unit = said[0];
    }
    if (t > 0 && unit < a_units)
      wait_until(p.progress, progress,
                 [&](uint32_t v) { return (v & kUpdated) == u_units * (uint32_t)t; }, &said[2]);
    while (unit < a_units) {
      const bool changed = __syncthreads_or(
          assign_points(p, unit * kWavesPerBlock + w, a_units * kWavesPerBlock, t));
      if (threadIdx.x == 0) {
        const uint32_t mark = kAssigned + (changed ? kChanged : 0u) + (claims ? kClaim : 0u);
        __threadfence();
        const uint32_t old = add_shared(word, mark);
        seen = old + mark;
        said[1] = old & kClaims;
      }
      __syncthreads();
      unit = claims ? said[1] : unit + expected;
    }
    const uint32_t all = wait_until(
        word, seen, [&](uint32_t v) { return (v / kAssigned & kUnits) == a_units; }, &said[2]);
    if (!any_change(all)) return;
    if (!claims) unit = a_units + blockIdx.x;
    while (unit < a_units + u_units) {
      update_centroids(p, (unit - a_units) * kWavesPerBlock + w, u_units * kWavesPerBlock, lists[w]);
      __syncthreads();
      if (threadIdx.x == 0) {
        __threadfence();
        progress = add_shared(p.progress, 1u) + 1u;
        if (claims) said[1] = add_shared(word, kClaim) & kClaims;
      }
      __syncthreads();
      unit = claims ? said[1] : unit + expected;
    }
  }
}

}  // namespace

size_t kmeans_workspace_bytes(int32_t m, int32_t max_iter) {
  return ((size_t)m + (size_t)max_iter) * sizeof(uint32_t);
}

int launch_kmeans(const float *features, int32_t n, int32_t dim, int32_t m, const uint32_t *init,
                  int32_t max_iter, uint32_t *assign, double *centroids, uint32_t *counts,
                  void *workspace, hipStream_t stream, int32_t persist_groups,
                  int32_t held_back) {
  // [m] seed textures (passed by value: word 0 the progress), then [max_iter] flags
  uint32_t *dinit = (uint32_t *)workspace;
  const Problem p = {features, n, dim, m, centroids, assign, counts, dinit + m, dinit, max_iter};
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
    const auto units_of = [&](int64_t waves) {
      return groups_of(waves) < kPersistGroups ? groups_of(waves) : (int64_t)kPersistGroups;
    };
    const int64_t a_units = units_of(n), u_units = units_of(units);
    const int64_t share = a_units > u_units ? a_units : u_units;
    int64_t groups = persist_groups;
    if (groups < 1) {
      int dev = 0, cus = 0;
      if (hipGetDevice(&dev) != hipSuccess ||
          hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return NTC_ERR_HIP;
      groups = share < cus ? share : cus;
    }
    if (groups > kPersistGroups) groups = kPersistGroups;
    hipLaunchKernelGGL(kmeans_persistent, dim3((unsigned)groups), dim3(kBlock), 0, stream, p,
                       (uint32_t)a_units, (uint32_t)u_units, (uint32_t)(groups + held_back));
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
