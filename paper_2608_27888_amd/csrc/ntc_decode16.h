// ntc_decode16.h -- binned decode on v_mfma_f32_16x16x32_f16 with an
// LDS-staged latent gather (gfx950).
//
// The decode of a 64-query tile of one bin (one decoder, the shared or
// clustered decoder of Sec. 1 and Sec. 4.4): latent sampling, then the MLP of
// ntc_decode_kernels.h, its weights staged in LDS.  The departure:
//
//  * Latent taps come from a wave-private LDS region instead of one 16-byte
//    global load per tap and lane.  A vector-memory instruction costs the CU
//    16 cycles of L1 return bandwidth for 64 lanes x 16 bytes whether or not
//    the lanes share addresses, and in binned order the 64 queries of a tile
//    touch about 13 distinct bilinear quads at the finest level (not 64): a
//    query whose quad differs from the previous lane's is a leader, each
//    leader's quad is fetched once by a few lanes (1-4 loads per level instead
//    of 8), written to LDS, and every lane reads its four taps from there.  The
//    fetch for tile k+1 is issued at the start of tile k into a few registers,
//    so its latency is hidden by a whole tile of work.  A level whose tile has
//    more leaders than the region holds is fetched tap by tap from memory for
//    that tile.
//
// Selected with NTC_GATHER_STAGED for binned decode without mip blending.  On
// MI355X it is slower than the direct gather of ntc_decode_kernels.h: the
// planning (leaders, slots, the exchange of quad addresses) adds about 40 VALU
// instructions per tile, and its plan and prefetches keep it at three waves per
// SIMD (pass over the 4K frame of 16 decoders 213 us against 185, over a 1080p one
// 75 against 61).
#pragma once

#include "ntc_decode_kernels.h"

namespace ntc {
namespace {

// ----------------------------------------------------------------- staging

// Wave-private LDS staging of the bilinear quads of one tile.  A quad is the
// 2x2 texels of one level around a query: 4 * CH / 8 pieces of 16 bytes,
// (x0, y0), (x0 + 1, y0), (x0, y0 + 1), (x0 + 1, y0 + 1), each texel's pieces
// in channel order.  Region of level l: cap(l) quad slots of QS bytes (a quad
// and 16 bytes of padding: the lanes of one read instruction address
// different slots at the same piece offset, and the padding spreads those
// slots over distinct LDS banks); then an exchange table of 8 bytes per slot
// (the quad's fp16 element offset).
template <int CH>
struct Staging {
  static constexpr int NV = CH / 8;          // pieces per texel
  static constexpr int PIECES = 4 * NV;      // pieces per quad
  static constexpr int QB = PIECES * 16;     // bytes per quad
  static constexpr int QS = QB + 16;         // bytes per slot
  static constexpr int loads(int l) { return l == 0 ? 4 : 3; }   // 16-byte loads per lane and level
  static constexpr int cap(int l) { return loads(l) * kWave / PIECES; }  // quads per level
  static constexpr int region(int l) {
    int b = 0;
    for (int i = 0; i < l; ++i) b += cap(i) * QS;
    return b;
  }
  template <int NL>
  static constexpr int bytes() {
    return region(NL) + xchg_bytes<NL>();
  }
  template <int NL>
  static constexpr int xchg_bytes() {
    int b = 0;
    for (int l = 0; l < NL; ++l) b += cap(l) * 8;
    return b;
  }
  template <int NL>
  static constexpr int xchg(int l) {
    int b = region(NL);
    for (int i = 0; i < l; ++i) b += cap(i) * 8;
    return b;
  }
  // LDS byte offset, inside its level's region, of piece 64 m + lane of the
  // level's staged quads (quad (64 m + lane) / PIECES, piece (64 m + lane) %
  // PIECES).
  static constexpr int piece_pos(int m, int lane) {
    return ((m * kWave + lane) / PIECES) * QS + ((m * kWave + lane) % PIECES) * 16;
  }
};

// Per-lane plan of one tile: for each level, the byte offset of the lane's
// quad in the wave's staging region (or of nothing when the level is fetched
// tap by tap) and its bilinear position; plus the query's texture and uv for
// such a level.
template <int NL>
struct TilePlan {
  uint32_t tap_off[NL];  // word offset in LDS of the lane's quad (staged levels)
  float fx[NL], fy[NL];
  uint32_t staged;       // wave-uniform: bit l set when level l is staged
};

// Global data of the leaders' quads of the next tile, in registers until they
// are written to LDS.
template <int NL>
struct StageData {
  u32x4 v[NL][4];
};

// Plans the tile whose (validated) query data is `qq`: bilinear positions,
// leaders (a valid query whose quad differs from the previous lane's, or whose
// previous lane holds no valid query), slots, and the loads of the leaders'
// quads into `sd` (issued, not waited for).  wave_w is the word offset of the
// wave's staging region in `lds`.  A wave's LDS operations execute in order,
// so the exchange table written and read back here needs no barrier.
template <int NL, int CH>
__device__ __forceinline__ TilePlan<NL> plan_tile(const DecodeArgs &a, const Query &qq,
                                                  uint32_t *lds, uint32_t wave_w,
                                                  const uint32_t (&piece_off)[NL],
                                                  StageData<NL> &sd) {
  using St = Staging<CH>;
  TilePlan<NL> P;
  P.staged = 0;
  const uint32_t lane = lane_id();
  // previous lane's texture and validity (lane 0 has none)
  const uint32_t valid = qq.valid ? 1u : 0u;
  const uint32_t prev_valid = __builtin_amdgcn_update_dpp(0u, valid, 0x138, 0xf, 0xf, false);
  const uint32_t prev_tex = __builtin_amdgcn_update_dpp(0u, qq.tex, 0x138, 0xf, 0xf, false);
  const bool new_run = qq.valid && (!prev_valid || prev_tex != qq.tex);
  const uint64_t tex_base = (uint64_t)qq.tex * (uint64_t)a.tex_stride;
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const float resf = a.resf[l];
    const float x = __builtin_fmaf(qq.u, resf, -0.5f), y = __builtin_fmaf(qq.v, resf, -0.5f);
    const float hi = resf - 2.f;
    const float x0 = __builtin_amdgcn_fmed3f(__builtin_floorf(x), 0.f, hi);
    const float y0 = __builtin_amdgcn_fmed3f(__builtin_floorf(y), 0.f, hi);
    P.fx[l] = __builtin_amdgcn_fmed3f(x - x0, 0.f, 1.f);
    P.fy[l] = __builtin_amdgcn_fmed3f(y - y0, 0.f, 1.f);
    const uint32_t idx = (uint32_t)y0 * (uint32_t)a.res[l] + (uint32_t)x0;
    const uint32_t prev_idx = __builtin_amdgcn_update_dpp(0u, idx, 0x138, 0xf, 0xf, false);
    const bool lead = new_run || (qq.valid && prev_idx != idx);
    const uint64_t mask = ballot(lead);
    const uint32_t nlead = (uint32_t)__builtin_popcountll(mask);
    // slot of the lane's leader (lanes before the first leader hold no valid query)
    const uint32_t rank = lanes_below(mask) + (lead ? 1u : 0u);
    const uint32_t slot = rank ? rank - 1u : 0u;
    P.tap_off[l] = wave_w + (St::region(l) + slot * St::QS) / 4;
    if (nlead <= (uint32_t)St::cap(l)) P.staged |= 1u << l;
    // The leaders' quad addresses (fp16 element offsets) go through the exchange
    // table; every load of the level is issued whatever the number of leaders
    // (no branch: a conditional load would be waited for right away), pieces
    // past the last leader's repeating its quad.  A level with more leaders than
    // the table holds is not staged; its loads only fill registers.
    uint64_t *xchg = (uint64_t *)(lds + wave_w + St::template xchg<NL>(l) / 4);
    const uint64_t elem = tex_base + a.level_off[l] + (uint64_t)idx * CH;
    // a wave without a valid query (no leader) has lane 0 enter texture 0's
    // first texels, which always exist; entries 0 .. last are written here
    if (nlead ? lead && slot < (uint32_t)St::cap(l) : lane == 0u) xchg[nlead ? slot : 0u] = nlead ? elem : 0ull;
    const uint32_t last = nlead ? min(nlead, (uint32_t)St::cap(l)) - 1u : 0u;
#pragma unroll
    for (int m = 0; m < St::loads(l); ++m) {
      const uint32_t k = min((m * kWave + lane) / St::PIECES, last);
      const char *src = (const char *)(a.latents + xchg[k]) + piece_off[l];
      sd.v[l][m] = *(const u32x4 *)src;
    }
  }
  return P;
}

// Writes the staged quads of a plan into the wave's region (after the wave is
// done reading the previous tile's taps from it).
template <int NL, int CH>
__device__ __forceinline__ void write_staged(const TilePlan<NL> &P, const StageData<NL> &sd,
                                             uint32_t *lds, uint32_t wave_w) {
  using St = Staging<CH>;
  const uint32_t lane = lane_id();
#pragma unroll
  for (int l = 0; l < NL; ++l) {
#pragma unroll
    for (int m = 0; m < St::loads(l); ++m)
      *(u32x4 *)(lds + wave_w + (St::region(l) + St::piece_pos(m, (int)lane)) / 4) = sd.v[l][m];
  }
}

// Features of the lane's query (lane = query slot) from the staged quads, or,
// for a level that was not staged, from taps loaded here.
template <int NL, int CH, int PE>
__device__ __forceinline__ void gather_staged(const DecodeArgs &a, const Query &qq,
                                              const TilePlan<NL> &P, const uint32_t *lds,
                                              uint32_t (&x)[(NL * CH + PE) / 2]) {
  using St = Staging<CH>;
  if constexpr (PE > 0) pos_encoding<PE>(qq.u, qq.v, x + NL * CH / 2);
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    LevelTaps<CH> L;
    if (P.staged & (1u << l)) {
      const u32x4 *q = (const u32x4 *)(lds + P.tap_off[l]);
#pragma unroll
      for (int i = 0; i < St::NV; ++i) {
        L.t00[i] = q[0 * St::NV + i];
        L.t10[i] = q[1 * St::NV + i];
        L.t01[i] = q[2 * St::NV + i];
        L.t11[i] = q[3 * St::NV + i];
      }
      L.fx = P.fx[l];
      L.fy = P.fy[l];
    } else {
      const uint16_t *tex = a.latents + (size_t)qq.tex * (size_t)a.tex_stride;
      fetch_level<CH>(tex, a.level_off[l], a.res[l], a.resf[l], qq.u, qq.v, L);
    }
    interp_level_h2<CH>(L, x + l * CH / 2);
  }
}

// ----------------------------------------------------------------- kernel

// Waves per workgroup and per SIMD of the 16x16 binned kernel.  64-wide decoders: one
// 12-wave workgroup per CU shares one staged decoder.  The MLP's activations, the next
// tile's plan and the query prefetches don't all fit the 168 VGPRs of three waves per
// SIMD (most forms spill 12-88 bytes a lane); two waves per SIMD spill nothing, but
// the 4K frame takes 222 us against 213 (1080p 74 against 75, two hidden layers 84
// against 88).  128-wide decoders use 8-wave workgroups, 2 waves per SIMD.
template <int HID>
constexpr int kWaves16 = HID > 64 ? 8 : 12;
template <int HID>
constexpr int kThreads16 = kWaves16<HID> * kWave;
template <int HID>
constexpr int kWavesPerEu16 = HID > 64 ? 2 : 3;

template <int NL, int CH, int PE, int HID, int NH, int STORE, bool LEAKY>
__global__ void __launch_bounds__((kThreads16<HID>), (kWavesPerEu16<HID>))
decode_binned16(const DecodeArgs a, uint32_t image_bytes) {
  constexpr int WAVES = kWaves16<HID>;
  constexpr int THREADS = kThreads16<HID>;
  constexpr bool WIDE = false;  // widths up to 8 only
  using S = Shape<NL, CH, PE, HID>;
  using N = Net<NL, CH, PE, HID, NH>;
  using St = Staging<CH>;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  const uint32_t w = threadIdx.x / kWave, lane = lane_id();
  const uint32_t D = (uint32_t)a.n_decoders;
  const __amdgpu_buffer_rsrc_t out_rsrc = out_resource(a);
  // this wave's staging region: a word offset in `lds`, past the decoder image
  const uint32_t wave_w = (image_bytes + w * (uint32_t)St::template bytes<NL>()) / 4;
  // byte offset of this lane's piece inside a quad, per level
  uint32_t piece_off[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const uint32_t p = lane % St::PIECES, tap = p / St::NV, vec = p % St::NV;
    piece_off[l] = (tap & 1u) * CH * 2u + (tap >> 1) * (uint32_t)a.res[l] * CH * 2u + vec * 16u;
  }
  const uint64_t slots = min((uint64_t)bin_off(a, D), a.perm_capacity);
  const uint32_t total_tiles = (uint32_t)(slots / kWave);
  const uint32_t per = (total_tiles + gridDim.x - 1) / gridDim.x;
  const uint32_t blk = xcd_local_block(blockIdx.x, gridDim.x);
  const uint32_t t = blk * per;
  const uint32_t t_end = min(t + per, total_tiles);
  if (t >= t_end) return;
  uint32_t lo = 0, hi = D;  // bin holding slot 64 t: bin_offset[lo] <= 64 t < bin_offset[hi]
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (bin_off(a, mid) <= t * kWave) lo = mid; else hi = mid;
  }
  Group g0 = group_at<WAVES>(a, t, lo, bin_off(a, lo + 1) / kWave, D, t_end);
  Group g1 = next_group<WAVES>(a, g0, D, t_end);
  Group g2 = next_group<WAVES>(a, g1, D, t_end);
  Group g3 = next_group<WAVES>(a, g2, D, t_end);
  struct Slot {
    uint32_t raw;
    bool has;
  };
  auto slot_query = [&](const Group &g) -> Slot {
    const bool has = w < g.n;
    return Slot{a.perm[has ? (g.t + w) * kWave + lane : 0u], has};
  };
  auto restage = [&](uint32_t d) {
    __syncthreads();
    stage_decoder<N, THREADS>(a, d, lds);
    __syncthreads();
  };
  // prologue: tile 0 planned and staged, tile 1's query data and tile 2's
  // permutation entry in flight
  const Slot s0 = slot_query(g0);
  Query cur = validate(a, load_query<NL, false>(a, s0.raw, s0.has));
  restage(g0.d);
  uint32_t staged_dec = g0.d;
  StageData<NL> sd;
  TilePlan<NL> plan = plan_tile<NL, CH>(a, cur, lds, wave_w, piece_off, sd);
  write_staged<NL, CH>(plan, sd, lds, wave_w);
  const Slot s1 = slot_query(g1);
  Query q_next = load_query<NL, false>(a, s1.raw, s1.has);
  Slot p_next = slot_query(g2);
  // the previous tile's output, stored one tile late (none before the first:
  // its stores are dropped, so every tile issues the same stores)
  TileOut<WIDE> pending;
#pragma unroll
  for (int i = 0; i < TileOut<WIDE>::G; ++i) {
    pending.v[i] = u32x4{0u, 0u, 0u, 0u};
    pending.q[i] = 0u;
  }
  pending.ok = 0u;
  auto tile = [&](const Query &q_in, const Slot &p_in, Query &q_out, Slot &p_out) {
    // prefetches: query data two tiles ahead, the permutation entry three ahead
    q_out = load_query<NL, false>(a, p_in.raw, p_in.has);
    p_out = slot_query(g3);
    __builtin_amdgcn_sched_barrier(0);
    // plan of the next tile; its quads' loads go out now
    const Query nxt = validate(a, q_in);
    const TilePlan<NL> plan_next = plan_tile<NL, CH>(a, nxt, lds, wave_w, piece_off, sd);
    __builtin_amdgcn_sched_barrier(0);
    // the previous tile's stores, after every load of this tile in issue order
    store_out16<STORE, WIDE>(out_rsrc, a.out_dim, pending, a.out_f16);
    __builtin_amdgcn_sched_barrier(0);
    // this tile: features from the staged quads
    uint32_t x[S::F / 2];
    gather_staged<NL, CH, PE>(a, cur, plan, lds, x);
    half8 xb[4][S::KS0];
    to_b16<S::KS0, S::F / 2>(x, xb);
    __builtin_amdgcn_sched_barrier(0);
    // the region is free now (this tile's taps are read): the next tile's quads go in
    write_staged<NL, CH>(plan_next, sd, lds, wave_w);
    floatx4 y[4];
    LdsNet<NL, CH, PE, HID, NH> net;
    net.lds = lds;
    mlp<NL, CH, PE, HID, NH, LEAKY>(net, xb, y, a.slope_h2);
    const float *ob = net.biases() + HID * (1 + NH);
    pending = finish16<WIDE>(y, ob, cur.q, cur.valid);
    __builtin_amdgcn_sched_barrier(0);
    if (g1.n && g1.d != staged_dec) {
      restage(g1.d);
      staged_dec = g1.d;
    }
    cur = nxt;
    plan = plan_next;
    g0 = g1;
    g1 = g2;
    g2 = g3;
    g3 = next_group<WAVES>(a, g3, D, t_end);
  };
  Query q_b;
  Slot p_b;
  for (;;) {
    if (!g0.n) break;
    tile(q_next, p_next, q_b, p_b);
    if (!g0.n) break;
    tile(q_b, p_b, q_next, p_next);
  }
  store_out16<STORE, WIDE>(out_rsrc, a.out_dim, pending, a.out_f16);
}

// LDS bytes of a decode_binned16 workgroup: the decoder image (16-byte
// aligned), then every wave's staging region.
template <int NL, int CH, int PE, int HID, int NH>
inline size_t binned16_lds_bytes(uint32_t *image_bytes) {
  const uint32_t ib = ((uint32_t)Net<NL, CH, PE, HID, NH>::kImageBytes + 15u) & ~15u;
  if (image_bytes) *image_bytes = ib;
  return (size_t)ib + (size_t)kWaves16<HID> * Staging<CH>::template bytes<NL>();
}

template <int NL, int CH, int PE, int HID, int NH, int STORE, bool LEAKY>
int launch_binned16(const DecodeArgs &a, hipStream_t stream) {
  uint32_t image_bytes = 0;
  const size_t lds = binned16_lds_bytes<NL, CH, PE, HID, NH>(&image_bytes);
  const void *fn = (const void *)decode_binned16<NL, CH, PE, HID, NH, STORE, LEAKY>;
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return NTC_ERR_HIP;
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess)
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  constexpr int threads = kThreads16<HID>;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  const uint64_t cap = (uint64_t)cus * (uint64_t)per_cu;
  uint64_t blocks = ((uint64_t)a.max_tiles + kWaves16<HID> - 1) / kWaves16<HID>;
  if (blocks > cap) blocks = cap;
  if (blocks == 0) return NTC_OK;
  hipLaunchKernelGGL((decode_binned16<NL, CH, PE, HID, NH, STORE, LEAKY>), dim3((unsigned)blocks),
                     dim3(threads), lds, stream, a, image_bytes);
  return hip_status(hipGetLastError());
}

}  // namespace
}  // namespace ntc
