// ntc_bins.hip -- stable counting sort of texel queries by decoder id.
//
// Groups the query stream so that every 64-slot tile of `perm` belongs to one
// decoder; a wave then evaluates a single decoder, the situation the paper's
// shared decoder creates (Sec. 1; Sec. 4.4 "Performance analysis").  The
// binning itself is not in the paper.
//
// The unit of the sort is one wave's contiguous slice of the query stream
// (slice g = workgroup * waves + wave), processed in batches of kBatchRows rows
// of 64 queries.
//
// Up to 64 decoders (while every workgroup can sum the rows of tot in two
// rounds of loads), two kernels on workgroups of 4 to 16 waves:
//   count : every wave resolves the decoder id of each query of its slice
//           (tex_to_dec[tex_id[q]]) and counts the ids; the workgroup writes its
//           sums over its waves, column b of tot[d][b] (row D: invalid
//           queries), and for slice g its waves' exclusive prefix, hist[d][g].
//   place : every workgroup sums the rows of tot (at most 512 words each): the
//           totals give the padded bin offsets (workgroup 0 writes bin_count
//           and bin_offset, the padding slots are shared out among the
//           workgroups), the columns before its own its offset inside every
//           bin, and hist[d][g] each wave's offset after that.  Each wave then
//           resolves the ids of its slice again and writes every query to the
//           next slot of its bin.
// Otherwise three kernels on workgroups of 4 waves: count writes hist only;
// scan (workgroup d) turns row d of hist into its exclusive prefix over slices
// and writes bin_count[d]; place scans bin_count into the padded offsets and
// starts its cursors at bin_offset[d] + hist[d][g].
// Inside a 64-query row the lanes that share a decoder id are ranked with
// ballots and lane counts (peel_row, match_row), so the order inside a bin is
// ascending query index and the permutation is unique.  With at
// most 64 decoders the wave's counters (count) and cursors (place) live in one
// register, lane k holding decoder k's, and a row costs no LDS access; with more
// they live in a wave-private LDS table.  A wave issues the id loads of a whole
// batch, then all of its map lookups, before it uses any of them.  The decoder
// ids are not stored between the passes: reading tex_id twice moves as many
// bytes as writing and reading back 16-bit ids, and leaves the count pass
// without stores.  Workgroups are numbered XCD by XCD, so the histogram
// entries of neighbouring slices are written from one L2.
#include "ntc_internal.h"

namespace ntc {
namespace {

constexpr int kBatchRows = 16;                                   // rows of 64 per wave batch
constexpr int64_t kWaveQuantum = (int64_t)kWave * kBatchRows;    // queries per wave batch
constexpr int64_t kTargetBlocks = 2048;                          // workgroups, at most
// The two-kernel path: workgroups of 4, 8 or 16 waves, at most kSumBlocks of
// them, so that every place workgroup can sum the tot rows.  The widest
// workgroups that still give every CU one (kCus) keep many waves in flight on a
// large frame; a smaller frame takes narrower ones, since the per-row ranking
// runs on the CU's one scalar unit and a CU without a workgroup sits idle.
constexpr int64_t kSumBlocks = 512;
constexpr int64_t kCus = 256;
constexpr int kSumLanes = 32;  // place: lanes per row of tot
constexpr int kSumPer = 16;    // place: words of a row per lane
constexpr int kSumRounds = 2;  // place: at most this many rounds of those loads
constexpr int64_t kMaxHistWords = (int64_t)1 << 20;              // slice histograms, at most
constexpr uint32_t kOutside = 0xFFFFFFFFu;                       // a lane past the slice
constexpr int kScanThreads = 1024;                               // scan: threads per column
constexpr int kScanPerThread = 8;                                // scan: slices per thread
constexpr uint32_t kRegDecoders = kWave;                         // register tables up to here

static_assert(kTargetBlocks * kWavesPerBlock <= (int64_t)kScanThreads * kScanPerThread,
              "one scan pass covers every slice");

// The workspace starts with kStatusWords status words -- [1] is the invalid
// query count -- followed by hist[n_decoders + 1][slices] and, on the
// two-kernel path, tot[n_decoders + 1][workgroups].
constexpr int kStatusWords = 4;

// Query range [beg, end) of wave w of a workgroup b of WAVES waves.
struct Slice {
  uint64_t beg, end;
};

template <int WAVES>
__device__ __forceinline__ Slice slice_of(uint32_t b, uint32_t w, uint64_t chunk, uint64_t n) {
  const uint64_t cbeg = (uint64_t)b * chunk;
  const uint64_t cend = cbeg + chunk < n ? cbeg + chunk : n;
  const uint64_t wchunk = chunk / WAVES;
  const uint64_t beg = cbeg + w * wchunk < cend ? cbeg + w * wchunk : cend;
  return Slice{beg, beg + wchunk < cend ? beg + wchunk : cend};
}

// Decoder ids of the batch of kBatchRows rows starting at query `base` (wave
// uniform, base < end): lanes at or past `end` get kOutside, invalid queries
// `invalid`.  Every id load is issued, then every map lookup, before any result
// is used; the loads are unconditional (clamped into the slice), addressed from
// one wave-uniform pointer with 32-bit lane offsets.  ANEW: the offsets are formed
// anew for every batch.  Where every row is matched a batch is one straight block,
// and the compiler would keep them from one to the next: 68-72 registers in count
// (of 16-wave workgroups one a CU instead of two) and spills in place (4K frame of
// two decoders, binning 31.3 us against 28.6).
template <bool ANEW>
__device__ __forceinline__ void load_batch(const uint32_t *__restrict__ tex_id,
                                           const uint32_t *__restrict__ tex_to_dec,
                                           uint32_t n_textures, uint32_t n_decoders,
                                           uint32_t invalid, uint64_t base, uint64_t end,
                                           uint32_t lane, uint32_t (&d)[kBatchRows]) {
  if constexpr (ANEW) asm volatile("" : "+v"(lane));
  const uint32_t *row = tex_id + base;
  const uint64_t left = end - base;
  const uint32_t lim = left < (uint64_t)kWaveQuantum ? (uint32_t)left : (uint32_t)kWaveQuantum;
#pragma unroll
  for (int j = 0; j < kBatchRows; ++j) {
    const uint32_t o = (uint32_t)j * kWave + lane;
    d[j] = row[o < lim - 1 ? o : lim - 1];
  }
  uint32_t m[kBatchRows];
#pragma unroll
  for (int j = 0; j < kBatchRows; ++j) m[j] = tex_to_dec[d[j] < n_textures ? d[j] : 0u];
#pragma unroll
  for (int j = 0; j < kBatchRows; ++j) {
    const uint32_t o = (uint32_t)j * kWave + lane;
    d[j] = o >= lim ? kOutside : d[j] < n_textures && m[j] < n_decoders ? m[j] : invalid;
  }
}

// A row of 64 queries is ranked by decoder in one of two ways, with the same
// result; the wave's table of one value per decoder (REG: lane k of `reg`, else
// word k of the wave's LDS table) advances by the row's counts.
//   peel : one pass per distinct decoder of the row (a ballot and a lane read),
//          15 instructions each, half of them on the CU's one scalar unit.
//   match: every lane finds the lanes with its decoder from ballots of the id's
//          B bits: 4 vector instructions a bit whatever the row holds, no scalar
//          chain.
// Rows of large screen regions hold one or two decoders, where peeling is faster
// (4K clustered frame, 16 decoders, 1.98 a row: 34.5 us against 41 for matching
// every row); rows of small tiles hold many (1080p, 64 decoders in 8x8 tiles, 7.6 a
// row: 30.2 us peeling, 19.8 matching).  So with more than 16 decoders the first
// row of a batch of 16 is peeled, and when it held more than kPeelMost decoders
// the other rows are matched.  With at most 4 decoders (2 bits) every row is
// matched (65,536 random queries of 2 decoders: 13.7 -> 11.7 us; 4K frames of regions
// as fast as peeling or 2 % slower: 25.6 us against 26.4 with two decoders, 29.1 against 28.5
// with four, where a peeled first row that decides takes 29.4 and 31.0); with 5 to 16
// every row is peeled (the choice alone cost the 4K clustered frame 2 us; 8x8 tiles of
// 16 decoders take 27.6 us at 1080p and 54.6 at 4K so, as before rows were matched).
constexpr uint32_t kPeelMost = 4;

// Lanes of `valid` whose value equals v, compared in its low B bits; v may differ
// per lane.  bal: ballots of those bits.
template <int B>
struct RowBits {
  uint64_t valid, bal[B > 0 ? B : 1];
  __device__ __forceinline__ RowBits(uint32_t d, uint64_t valid_lanes) : valid(valid_lanes) {
#pragma unroll
    for (int b = 0; b < B; ++b) bal[b] = ballot((d >> b) & 1u);
  }
  __device__ __forceinline__ uint64_t equal(uint32_t v) const {
    uint32_t lo = (uint32_t)valid, hi = (uint32_t)(valid >> 32);
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)v, b, 1);  // all ones or zero
      lo &= ~((uint32_t)bal[b] ^ m);
      hi &= ~((uint32_t)(bal[b] >> 32) ^ m);
    }
    return (uint64_t)hi << 32 | lo;
  }
};

__device__ __forceinline__ uint32_t popcount64(uint64_t m) {
  return (uint32_t)__builtin_popcountll(m);
}

// Number of decoder-id bits the row functions are compiled for: the next of
// these that holds D ids, or with LDS tables D + 1 (id D counts the invalid).
constexpr int id_bits(uint32_t D) {
  return D <= 1 ? 0 : D <= 2 ? 1 : D <= 4 ? 2 : D <= 16 ? 4 : D <= 64 ? 6 : D < 256 ? 8
         : D < 1024 ? 10 : 13;
}
constexpr bool peels(int bits) { return bits > 2; }
constexpr bool matches(int bits) { return bits <= 2 || bits > 4; }

// d: decoder ids, kOutside for a lane that does not count.  RANK: returns each
// lane's slot, its decoder's value plus the number of lanes below it with the
// same decoder.  (The LDS operations of a wave execute in order, so rows take
// their values in order.)
template <bool REG, bool RANK>
__device__ __forceinline__ uint32_t peel_row(uint32_t d, uint32_t &reg, uint32_t *table,
                                             uint32_t lane, uint32_t &distinct) {
  uint64_t todo = ballot(d != kOutside);
  uint32_t pos = 0;
  distinct = 0;
  while (todo) {
    const uint32_t leader = (uint32_t)__builtin_ctzll(todo);
    const uint32_t dl = read_lane(d, leader);
    const uint64_t same = ballot(d == dl) & todo;
    const uint32_t c = popcount64(same);
    if constexpr (REG) {
      if constexpr (RANK) {
        const uint32_t at = read_lane(reg, dl);
        pos = d == dl ? at + lanes_below(same) : pos;
      }
      reg += lane == dl ? c : 0u;
    } else if constexpr (RANK) {  // the leader's returning atomic reads and advances
      uint32_t old = 0;
      if (lane == leader) old = atomicAdd(&table[dl], c);
      pos = d == dl ? read_lane(old, leader) + lanes_below(same) : pos;
    } else if (lane == leader) {
      atomicAdd(&table[dl], c);
    }
    todo &= ~same;
    ++distinct;
  }
  return pos;
}

template <bool REG, bool RANK, int B>
__device__ __forceinline__ uint32_t match_row(uint32_t d, uint32_t &reg, uint32_t *table,
                                              uint32_t lane) {
  const RowBits<B> row(d, ballot(d != kOutside));
  if constexpr (REG && !RANK) {
    reg += popcount64(row.equal(lane));
    return 0;
  } else {
    const uint64_t same = row.equal(d);
    const uint32_t rank = lanes_below(same);
    uint32_t at = 0;
    if constexpr (REG) {
      at = B == 0 ? read_lane(reg, 0)
                  : (uint32_t)__builtin_amdgcn_ds_bpermute((int)(d << 2), (int)reg);
      reg += popcount64(row.equal(lane));
    } else {
      uint32_t old = 0;  // the first lane of each decoder reads and advances its value
      if (d != kOutside && rank == 0) old = atomicAdd(&table[d], popcount64(same));
      if constexpr (RANK) {
        const uint32_t lo = (uint32_t)same, hi = (uint32_t)(same >> 32) | 1u << 31;
        const uint32_t first =
            lo ? (uint32_t)__builtin_ctz(lo) : 32u + (uint32_t)__builtin_ctz(hi);
        at = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(first << 2), (int)old);
      }
    }
    return at + rank;
  }
}

// The rows of a batch, peeled or matched; emit(j, slot) for every row j (RANK).
template <bool REG, bool RANK, int B, typename Emit>
__device__ __forceinline__ void batch_rows(const uint32_t (&d)[kBatchRows], uint32_t &reg,
                                           uint32_t *table, uint32_t lane, Emit emit) {
  if constexpr (REG && B == 1) {
    // Two decoders (ids 0 and 1): their values in scalar registers.  A row that
    // reads them from lanes of `reg` waits for the row before: binning and decode of
    // 41,400 queries 28.1 -> 27.2 us, binning of 2255 x 1273 16.5 -> 15.4, of 4K 26.8 ->
    // 25.6.
    uint32_t c0 = read_lane(reg, 0), c1 = read_lane(reg, 1);
#pragma unroll
    for (int j = 0; j < kBatchRows; ++j) {
      const uint64_t zeros = ballot(d[j] == 0), ones = ballot(d[j] == 1);
      if constexpr (RANK)
        emit(j, d[j] == 1 ? c1 + lanes_below(ones) : c0 + lanes_below(zeros));
      c0 += popcount64(zeros);
      c1 += popcount64(ones);
      __builtin_amdgcn_sched_barrier(0);  // else the rows' ballots fill the scalar registers
    }
    reg = lane == 0 ? c0 : lane == 1 ? c1 : reg;
    return;
  }
  constexpr int kFirst = peels(B) && matches(B) ? 1 : 0;
  uint32_t distinct = kPeelMost + 1, unused;
  if constexpr (kFirst) emit(0, peel_row<REG, RANK>(d[0], reg, table, lane, distinct));
  if constexpr (matches(B)) {
    if (distinct > kPeelMost) {
#pragma unroll
      for (int j = kFirst; j < kBatchRows; ++j)
        emit(j, match_row<REG, RANK, B>(d[j], reg, table, lane));
      return;
    }
  }
  if constexpr (peels(B)) {
#pragma unroll
    for (int j = kFirst; j < kBatchRows; ++j)
      emit(j, peel_row<REG, RANK>(d[j], reg, table, lane, unused));
  }
}

// REG: register tables (n_decoders <= 64).  tot (REG only): the workgroup's
// sums over its waves, column b of tot[n_decoders + 1][gridDim.x], with hist
// holding each wave's exclusive prefix over the workgroup's waves; NULL: hist
// holds each wave's own counts.  Eight waves per SIMD, asked for: with two decoders the
// rows' masks would take 106 scalar registers (4K frame 26.7 us, 25.6 at 78).
template <bool REG, int WAVES, int B>
__global__ void __launch_bounds__(WAVES * kWave) __attribute__((amdgpu_waves_per_eu(8)))
bins_count(const uint32_t *__restrict__ tex_id, uint32_t n,
           const uint32_t *__restrict__ tex_to_dec, uint32_t n_textures, uint32_t n_decoders,
           uint32_t chunk, uint32_t *__restrict__ hist, uint32_t *__restrict__ tot) {
  extern __shared__ uint32_t lds[];  // !REG: WAVES x (n_decoders + 1) counters
  __shared__ uint32_t part[REG ? WAVES : 1][kWave + 1];
  const uint32_t b = xcd_local_block(blockIdx.x, gridDim.x), lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t cols = n_decoders + 1, n_slices = gridDim.x * WAVES;
  const Slice sl = slice_of<WAVES>(b, w, chunk, n);
  uint32_t counts = 0, *table = lds + w * cols;
  if constexpr (!REG)
    for (uint32_t i = lane; i < cols; i += kWave) table[i] = 0;
  // With the register table the invalid queries are counted apart, in a
  // wave-uniform counter, so that all 64 lanes can hold decoders.
  uint32_t invalid = 0;
  for (uint64_t base = sl.beg; base < sl.end; base += kWaveQuantum) {
    uint32_t d[kBatchRows];
    load_batch<!peels(B)>(tex_id, tex_to_dec, n_textures, n_decoders, n_decoders, base, sl.end,
                          lane, d);
    if constexpr (REG) {
#pragma unroll
      for (int j = 0; j < kBatchRows; ++j) {
        const bool bad = d[j] == n_decoders;
        invalid += popcount64(ballot(bad));
        d[j] = bad ? kOutside : d[j];
      }
    }
    batch_rows<REG, false, B>(d, counts, table, lane, [](int, uint32_t) {});
  }
  if constexpr (REG) {
    const size_t col = b * WAVES + w;
    if (!tot) {
      if (lane < n_decoders) hist[(size_t)lane * n_slices + col] = counts;
      if (lane == 0) hist[(size_t)n_decoders * n_slices + col] = invalid;
    } else {
      part[w][lane] = counts;
      if (lane == 0) part[w][kWave] = invalid;
      __syncthreads();
      if (lane < n_decoders) {
        uint32_t excl = 0;
        for (uint32_t k = 0; k < w; ++k) excl += part[k][lane];
        hist[(size_t)lane * n_slices + col] = excl;
      }
      if (threadIdx.x < cols) {
        const uint32_t r = threadIdx.x < n_decoders ? threadIdx.x : kWave;
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) sum += part[k][r];
        tot[(size_t)threadIdx.x * gridDim.x + b] = sum;
      }
    }
  } else {
    // the workgroup's WAVES slices are neighbours in every row of hist: thread
    // t writes row t / WAVES, slice t % WAVES, so a wave covers 64 / WAVES rows
    // with pieces of 4 WAVES bytes
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < cols * WAVES; i += WAVES * kWave) {
      const uint32_t r = i / WAVES, ww = i % WAVES;
      hist[(size_t)r * n_slices + b * WAVES + ww] = lds[ww * cols + r];
    }
  }
}

// Exclusive scan over the workgroup of one value per thread; returns the total.
// tmp: one LDS word per wave.
template <int WAVES>
__device__ uint32_t block_exclusive_scan(uint32_t v, uint32_t &excl, uint32_t *tmp) {
  const uint32_t lane = lane_id(), w = threadIdx.x / kWave;
  uint32_t incl = v;
#pragma unroll
  for (int s = 1; s < kWave; s <<= 1) {
    const uint32_t o = __shfl_up(incl, s, kWave);
    if (lane >= (uint32_t)s) incl += o;
  }
  if (lane == kWave - 1) tmp[w] = incl;
  __syncthreads();
  uint32_t base = 0, total = 0;
#pragma unroll
  for (int k = 0; k < WAVES; ++k) {
    const uint32_t t = tmp[k];
    base += k < (int)w ? t : 0u;
    total += t;
  }
  __syncthreads();
  excl = base + incl - v;
  return total;
}

// Workgroup d scans row d of hist[cols][n_slices]; thread i owns slices
// [i * kScanPerThread, ...) and loads all of them at once.
__global__ void __launch_bounds__(kScanThreads)
bins_scan(uint32_t *__restrict__ hist, uint32_t n_slices, uint32_t n_decoders,
          uint32_t *__restrict__ bin_count, uint32_t *__restrict__ status,
          uint32_t *__restrict__ invalid_out) {
  __shared__ uint32_t tmp[kScanThreads / kWave];
  const uint32_t d = blockIdx.x;
  const uint32_t s0 = threadIdx.x * kScanPerThread;
  uint32_t *row = hist + (size_t)d * n_slices;
  uint32_t v[kScanPerThread];
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < kScanPerThread; ++k) {
    v[k] = s0 + k < n_slices ? row[s0 + k] : 0u;
    sum += v[k];
  }
  uint32_t excl;
  const uint32_t total = block_exclusive_scan<kScanThreads / kWave>(sum, excl, tmp);
#pragma unroll
  for (int k = 0; k < kScanPerThread; ++k) {
    if (s0 + k < n_slices) row[s0 + k] = excl;
    excl += v[k];
  }
  if (threadIdx.x == 0) {
    if (d < n_decoders) {
      bin_count[d] = total;
    } else {
      status[1] = total;
      if (invalid_out) *invalid_out = total;
    }
  }
}

// Place of the three-kernel path.
template <bool REG, int B>
__global__ void __launch_bounds__(kBlock)
bins_place(const uint32_t *__restrict__ tex_id, uint32_t n,
           const uint32_t *__restrict__ tex_to_dec, uint32_t n_textures, uint32_t n_decoders,
           uint32_t align, uint32_t chunk, const uint32_t *__restrict__ hist,
           const uint32_t *__restrict__ bin_count, uint32_t *__restrict__ bin_offset,
           uint32_t *__restrict__ perm) {
  extern __shared__ uint32_t lds[];  // kWavesPerBlock x n_decoders cursors
  __shared__ uint32_t scan_tmp[kWavesPerBlock];
  const uint32_t D = n_decoders;
  const uint32_t b = xcd_local_block(blockIdx.x, gridDim.x), lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t nblocks = gridDim.x, n_slices = nblocks * kWavesPerBlock;
  const Slice sl = slice_of<kWavesPerBlock>(b, w, chunk, n);
  // The first batch's ids are in flight during the offset scan below; invalid
  // queries are marked as outside: they go nowhere.
  uint32_t d[kBatchRows];
  if (sl.beg < sl.end)
    load_batch<!peels(B)>(tex_id, tex_to_dec, n_textures, D, kOutside, sl.beg, sl.end, lane, d);
  // Padded bin offsets: thread i owns decoders [dlo, dhi).
  const uint32_t dper = (D + kBlock - 1) / kBlock;
  const uint32_t dlo = min(threadIdx.x * dper, D);
  const uint32_t dhi = min(dlo + dper, D);
  uint32_t psum = 0;
  for (uint32_t k = dlo; k < dhi; ++k) psum += (bin_count[k] + align - 1) & ~(align - 1);
  uint32_t off;
  const uint32_t total = block_exclusive_scan<kWavesPerBlock>(psum, off, scan_tmp);
  // the slices' prefixes of decoder k: one 16-byte piece (n_slices is a
  // multiple of 4 and hist 16-byte aligned)
  static_assert(kWavesPerBlock == 4, "one 16-byte piece per decoder");
  const uint32_t *prefix = hist + b * kWavesPerBlock;
  for (uint32_t k = dlo; k < dhi; ++k) {
    const uint32_t cnt = bin_count[k];
    const uint32_t padded = (cnt + align - 1) & ~(align - 1);
    const uint4 p = *(const uint4 *)(prefix + (size_t)k * n_slices);
    lds[0 * D + k] = off + p.x;
    lds[1 * D + k] = off + p.y;
    lds[2 * D + k] = off + p.z;
    lds[3 * D + k] = off + p.w;
    if (b == 0) bin_offset[k] = off;
    if (k % nblocks == b)  // the padding slots of bin k
      for (uint32_t s = off + cnt; s < off + padded; ++s) perm[s] = NTC_PAD;
    off += padded;
  }
  if (b == 0 && threadIdx.x == 0) bin_offset[D] = total;
  __syncthreads();
  uint32_t *table = lds + w * D;
  uint32_t cursors = REG && lane < D ? table[lane] : 0u;
  for (uint64_t base = sl.beg; base < sl.end; base += kWaveQuantum) {
    if (base != sl.beg)
      load_batch<!peels(B)>(tex_id, tex_to_dec, n_textures, D, kOutside, base, sl.end, lane, d);
    batch_rows<REG, true, B>(d, cursors, table, lane, [&](int j, uint32_t pos) {
      if (d[j] != kOutside) perm[pos] = (uint32_t)(base + (uint64_t)j * kWave + lane);
    });
  }
}

// Place of the two-kernel path (register tables, n_decoders <= 64): the offsets
// come from tot and from this workgroup's columns of hist.
// Eight waves per SIMD (with 16-wave workgroups two per CU), so every
// workgroup of a 4K frame is resident at once (the scalar registers decide).
template <int WAVES, int B>
__global__ void __launch_bounds__(WAVES * kWave) __attribute__((amdgpu_waves_per_eu(8)))
bins_place_sum(const uint32_t *__restrict__ tex_id, uint32_t n,
               const uint32_t *__restrict__ tex_to_dec, uint32_t n_textures,
               uint32_t n_decoders, uint32_t align, uint32_t chunk,
               const uint32_t *__restrict__ hist, const uint32_t *__restrict__ tot,
               uint32_t *__restrict__ bin_count, uint32_t *__restrict__ bin_offset,
               uint32_t *__restrict__ perm, uint32_t *__restrict__ status,
               uint32_t *__restrict__ invalid_out) {
  __shared__ uint32_t total[kWave + 1], before[kWave + 1], start[kWave];
  const uint32_t D = n_decoders;
  const uint32_t b = xcd_local_block(blockIdx.x, gridDim.x), lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t nblocks = gridDim.x, n_slices = nblocks * WAVES;
  const Slice sl = slice_of<WAVES>(b, w, chunk, n);
  // The first batch's ids are in flight while the offsets are summed; invalid
  // queries are marked as outside: they go nowhere.
  uint32_t d[kBatchRows];
  if (sl.beg < sl.end)
    load_batch<!peels(B)>(tex_id, tex_to_dec, n_textures, D, kOutside, sl.beg, sl.end, lane, d);
  // Row r of tot (r = D: invalid queries): its total and its sum over the
  // workgroups before this one.  kSumLanes lanes take a row, kSumPer words
  // each, all loaded at once.
  static_assert(kSumLanes * kSumPer >= kSumBlocks, "a row fits its lanes");
  for (uint32_t t = threadIdx.x; t < kSumLanes * (D + 1); t += WAVES * kWave) {
    const uint32_t r = t / kSumLanes, i0 = (t % kSumLanes) * kSumPer;
    const uint32_t *row = tot + (size_t)r * nblocks;
    uint32_t v[kSumPer];
#pragma unroll
    for (int k = 0; k < kSumPer; ++k) v[k] = i0 + k < nblocks ? row[i0 + k] : 0u;
    uint32_t all = 0, prior = 0;
#pragma unroll
    for (int k = 0; k < kSumPer; ++k) {
      all += v[k];
      prior += i0 + k < b ? v[k] : 0u;
    }
    // the kSumLanes lanes of a row are one aligned group, all active
#pragma unroll
    for (int sh = kSumLanes / 2; sh > 0; sh >>= 1) {
      all += __shfl_xor(all, sh, kWave);
      prior += __shfl_xor(prior, sh, kWave);
    }
    const uint32_t k = r < D ? r : kWave;
    if (t % kSumLanes == 0) {
      total[k] = all;
      before[k] = prior;
    }
  }
  __syncthreads();
  if (w == 0) {
    // padded bin offsets: lane k holds decoder k
    const uint32_t cnt = lane < D ? total[lane] : 0u;
    const uint32_t padded = (cnt + align - 1) & ~(align - 1);
    uint32_t incl = padded;
#pragma unroll
    for (int s = 1; s < kWave; s <<= 1) {
      const uint32_t o = __shfl_up(incl, s, kWave);
      if (lane >= (uint32_t)s) incl += o;
    }
    const uint32_t off = incl - padded;
    start[lane] = off;
    if (b == 0) {
      if (lane < D) {
        bin_count[lane] = cnt;
        bin_offset[lane] = off;
      }
      if (lane == kWave - 1) {
        bin_offset[D] = incl;
        status[1] = total[kWave];
        if (invalid_out) *invalid_out = total[kWave];
      }
    }
    if (lane < D && lane % nblocks == b)  // the padding slots of bin `lane`
      for (uint32_t s = off + cnt; s < off + padded; ++s) perm[s] = NTC_PAD;
  }
  __syncthreads();
  // this wave's cursor of decoder k (lane k): the bin's offset, the queries of
  // the workgroups before this one, then those of this workgroup's earlier waves
  uint32_t cursors = 0;
  if (lane < D) cursors = start[lane] + before[lane] + hist[(size_t)lane * n_slices + b * WAVES + w];
  for (uint64_t base = sl.beg; base < sl.end; base += kWaveQuantum) {
    if (base != sl.beg)
      load_batch<!peels(B)>(tex_id, tex_to_dec, n_textures, D, kOutside, base, sl.end, lane, d);
    batch_rows<true, true, B>(d, cursors, nullptr, lane, [&](int j, uint32_t pos) {
      if (d[j] != kOutside) perm[pos] = (uint32_t)(base + (uint64_t)j * kWave + lane);
    });
  }
}

// Arguments of one binning.
struct BinsCall {
  const uint32_t *tex_id, *tex_to_dec;
  uint32_t n, n_textures, D, align, chunk;
  uint32_t *hist, *tot, *bin_count, *bin_offset, *perm, *status, *invalid_out;
  dim3 grid;
  hipStream_t stream;
};

// The two kernels of the register-table path, on workgroups of WAVES waves.
template <int WAVES, int B>
void launch_sum(const BinsCall &c) {
  const dim3 block(WAVES * kWave);
  hipLaunchKernelGGL((bins_count<true, WAVES, B>), c.grid, block, 0, c.stream, c.tex_id, c.n,
                     c.tex_to_dec, c.n_textures, c.D, c.chunk, c.hist, c.tot);
  hipLaunchKernelGGL((bins_place_sum<WAVES, B>), c.grid, block, 0, c.stream, c.tex_id, c.n,
                     c.tex_to_dec, c.n_textures, c.D, c.align, c.chunk, c.hist, c.tot, c.bin_count,
                     c.bin_offset, c.perm, c.status, c.invalid_out);
}

template <int B>
void launch_sum_waves(const BinsCall &c, int waves) {
  if (waves == 16) launch_sum<16, B>(c);
  else if (waves == 8) launch_sum<8, B>(c);
  else launch_sum<4, B>(c);
}

// Lets a kernel use more than the default 64 KB of dynamic LDS.
int allow_lds(const void *kernel, size_t bytes) {
  if (bytes + 64 <= 64 * 1024) return NTC_OK;
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) ==
                 hipSuccess
             ? NTC_OK
             : NTC_ERR_HIP;
}

// The three kernels.
template <bool REG, int B>
int launch_three(const BinsCall &c) {
  const size_t lds_count = REG ? 0 : (size_t)kWavesPerBlock * (c.D + 1) * sizeof(uint32_t);
  const size_t lds_place = (size_t)kWavesPerBlock * c.D * sizeof(uint32_t);
  int st = allow_lds((const void *)bins_count<REG, kWavesPerBlock, B>, lds_count);
  if (st == NTC_OK) st = allow_lds((const void *)bins_place<REG, B>, lds_place);
  if (st != NTC_OK) return st;
  const dim3 block(kBlock);
  hipLaunchKernelGGL((bins_count<REG, kWavesPerBlock, B>), c.grid, block, lds_count, c.stream,
                     c.tex_id, c.n, c.tex_to_dec, c.n_textures, c.D, c.chunk, c.hist, nullptr);
  hipLaunchKernelGGL(bins_scan, dim3(c.D + 1), dim3(kScanThreads), 0, c.stream, c.hist,
                     c.grid.x * kWavesPerBlock, c.D, c.bin_count, c.status, c.invalid_out);
  hipLaunchKernelGGL((bins_place<REG, B>), c.grid, block, lds_place, c.stream, c.tex_id, c.n,
                     c.tex_to_dec, c.n_textures, c.D, c.align, c.chunk, c.hist, c.bin_count,
                     c.bin_offset, c.perm);
  return NTC_OK;
}

}  // namespace

// Workgroups and queries per workgroup for chunks of multiples of
// kWaveQuantum * waves, at most max_blocks workgroups.
static void split(BinsLayout &L, int64_t n, int64_t max_blocks) {
  const int64_t quantum = kWaveQuantum * L.waves;
  int64_t chunk = (n + max_blocks - 1) / max_blocks;
  chunk = (chunk + quantum - 1) / quantum * quantum;
  if (chunk < quantum) chunk = quantum;
  L.chunk = chunk;
  L.blocks = n > 0 ? (n + chunk - 1) / chunk : 1;
}

BinsLayout bins_layout(int64_t n, int32_t n_decoders) {
  BinsLayout L;
  L.reg = (uint32_t)n_decoders <= kRegDecoders;
  L.sum = false;
  if (L.reg) {
    // the two-kernel path while a place workgroup sums the tot rows in at most
    // kSumRounds rounds of loads (kSumLanes threads per row)
    L.waves = n >= kCus * 16 * kWaveQuantum ? 16 : n >= kCus * 8 * kWaveQuantum ? 8 : 4;
    split(L, n, kSumBlocks);
    L.sum = (int64_t)kSumLanes * (n_decoders + 1) <= (int64_t)kSumRounds * L.waves * kWave;
  }
  if (!L.sum) {
    // fewer, longer slices for many decoders: the histograms stay within 4 MiB
    L.waves = kWavesPerBlock;
    int64_t max_blocks = kMaxHistWords / ((int64_t)kWavesPerBlock * (n_decoders + 1));
    max_blocks = max_blocks < 1 ? 1 : max_blocks > kTargetBlocks ? kTargetBlocks : max_blocks;
    split(L, n, max_blocks);
  }
  L.hist_words = (size_t)(n_decoders + 1) * (size_t)L.blocks * L.waves;
  L.tot_words = L.sum ? (size_t)(n_decoders + 1) * (size_t)L.blocks : 0;
  L.bytes = (kStatusWords + L.hist_words + L.tot_words) * sizeof(uint32_t);
  return L;
}

int launch_build_bins(const uint32_t *tex_id, int64_t n, const uint32_t *tex_to_dec,
                      int32_t n_textures, int32_t n_decoders, int32_t align,
                      uint32_t *bin_count, uint32_t *bin_offset, uint32_t *perm,
                      void *workspace, uint32_t *invalid_out, hipStream_t stream) {
  const BinsLayout L = bins_layout(n, n_decoders);
  uint32_t *status = (uint32_t *)workspace;
  uint32_t *hist = status + kStatusWords;
  const uint32_t D = (uint32_t)n_decoders;
  const BinsCall c = {tex_id, tex_to_dec, (uint32_t)n, (uint32_t)n_textures, D, (uint32_t)align,
                      (uint32_t)L.chunk, hist, hist + L.hist_words, bin_count, bin_offset, perm,
                      status, invalid_out, dim3((unsigned)L.blocks), stream};
  int st = NTC_OK;
  switch (id_bits(D)) {
    case 0: L.sum ? launch_sum_waves<0>(c, L.waves) : (void)(st = launch_three<true, 0>(c)); break;
    case 1: L.sum ? launch_sum_waves<1>(c, L.waves) : (void)(st = launch_three<true, 1>(c)); break;
    case 2: L.sum ? launch_sum_waves<2>(c, L.waves) : (void)(st = launch_three<true, 2>(c)); break;
    case 4: L.sum ? launch_sum_waves<4>(c, L.waves) : (void)(st = launch_three<true, 4>(c)); break;
    case 6: L.sum ? launch_sum_waves<6>(c, L.waves) : (void)(st = launch_three<true, 6>(c)); break;
    case 8: st = launch_three<false, 8>(c); break;
    case 10: st = launch_three<false, 10>(c); break;
    default: st = launch_three<false, 13>(c); break;
  }
  return st != NTC_OK ? st : hip_status(hipGetLastError());
}

size_t bins_status_bytes() { return kStatusWords * sizeof(uint32_t); }

int read_invalid_count(const void *workspace, uint64_t *n_invalid, hipStream_t stream) {
  const uint32_t *status = (const uint32_t *)workspace;
  uint32_t v = 0;
  hipError_t e = hipMemcpyAsync(&v, status + 1, sizeof(v), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return NTC_ERR_HIP;
  if (n_invalid) *n_invalid = v;
  return v ? NTC_ERR_INDEX : NTC_OK;
}

}  // namespace ntc
