#pragma once
// ntc_decode_kernels.h -- fused latent gather + MLP decoder on MFMA (gfx950).
//
// A query samples its texture's latent grid level by level (bilinear, texel
// centres at (i + 1/2)/res, clamp-to-edge; blended between levels by mip),
// concatenates the samples and runs an MLP decoder: ReLU hidden layers and a
// sigmoid output (Sec. 1 and Sec. 4 setup of the paper).  Tensor instructions
// run once per wave, so a wave whose queries use k decoders pays k MLP passes
// (Sec. 1, Sec. 4.4); binned mode feeds each wave one decoder.
//
// Work unit: one wave, one tile of 64 queries (lane l owns query slot l).
//
// Layer math: the layer output H^T = W X^T is computed with
// v_mfma_f32_16x16x32_f16, weights as the A operand (rows = output units) and
// the activations of 16 queries as the B operand (columns = queries); a tile is
// four such column blocks.  Lane l = (g = l / 16, n = l % 16): the B operand of
// column block j (queries 16j .. 16j+15) holds K-values 8g .. 8g+7 of query
// 16j + n, the A operand row n with the same K-values, the accumulator rows
// 4g .. 4g+3 of column n.  Converted to fp16, the accumulators of row blocks 2t
// and 2t+1 are directly the next layer's B operand for K-step t once that
// layer's weight columns are permuted (position 8g + e reads unit 32t + 4g + e
// for e < 4 and 32t + 16 + 4g + e - 4 otherwise); the permutation is applied
// when the weights are loaded, so activations never leave registers.  Biases
// are the accumulator input of the first MFMA of each row block.  Every kernel
// runs this one function (mlp), so binned and stream mode give the same bits.
//
// What bounds it: issue.  On the 4K clustered frame a tile takes 56 MFMAs (35 % of the
// SIMD's cycles) and 339 other vector instructions (53 % at one per 4 cycles), and the
// waves wait on a dependency or counter for 52 % of theirs (SQ counters).
// Why 16x16x32: it moves half the accumulator bytes per flop of 32x32x16 and pads an
// 8-wide output layer to 16 rows instead of 32: 161 -> 153 us on the 4K clustered
// frame, 50.7 -> 48 us on the 1080p one.
//
// Binned, a workgroup stages its decoder in LDS and every wave reads the fragments
// there: four waves per SIMD for 64-wide decoders (LDS image about 15 KB), two for
// 128-wide ones (84 fragments for 48-128-128-128-8, one image per CU).  Weights held in
// registers (14 fragments of 4 registers for 32-64-64-8) leave two waves per SIMD, too
// few wherever a tile does more between its MFMAs: at 1080p, 16 decoders, 2 x 8
// channels with mip 70.4 us against 61.9 from LDS, fp16 RGB rows with LeakyReLU 72.5
// against 64.1, two hidden layers 80.6 against 72.4; equal on the 4K clustered frame
// (185).  In stream order, where each wave takes its own decoders, 64-wide ones are
// held in registers.
//
// A second engine (decode_fma, end of the file) evaluates the MLP per lane with
// vector dot products instead: the paper's Non-Shared FMA comparison.
#include "ntc_internal.h"

namespace ntc {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef short short2v __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;

// Two floats -> packed fp16 pair, round to nearest even (one v_cvt_pk_f16_f32).
__device__ __forceinline__ uint32_t pack_half2(float a, float b) {
  const float2v f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, half2v));
}

__device__ __forceinline__ half8 as_half8(u32x4 v) { return __builtin_bit_cast(half8, v); }

__device__ __forceinline__ floatx4 mfma16(half8 a, half8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

template <int NL, int CH, int PE, int HID>
struct Shape {
  static constexpr int FL = NL * CH;         // latent features per query
  static constexpr int F = FL + PE;          // + positional-encoding features
  static constexpr int KS0 = (F + 31) / 32;  // 32-wide K-steps of layer 0 (zero padded)
  static constexpr int MB = HID / 16;        // 16-row blocks of a hidden layer
  static constexpr int KSH = HID / 32;       // K-steps of a layer fed by a hidden layer
  static_assert(F % 16 == 0, "feature count must be a multiple of 16");
  static_assert(HID % 32 == 0, "hidden width must be a multiple of 32");
  static_assert(CH == 8 || CH == 16, "8 or 16 channels per level");
  static_assert(PE % 16 == 0, "positional features come in whole 16-byte pieces");
};

// One decoder as A fragments (64 lanes x 16 bytes each: layer 0 by row block,
// then K-step; every hidden layer the same; the output layer's one row block)
// and fp32 biases (HID per hidden activation, then 16 of the output layer).
template <int NL, int CH, int PE, int HID, int NH>
struct Net {
  using S = Shape<NL, CH, PE, HID>;
  static constexpr int kHidden0 = S::MB * S::KS0;                // first hidden fragment
  static constexpr int kOut0 = kHidden0 + NH * S::MB * S::KSH;   // first output fragment
  static constexpr int kFrags = kOut0 + S::KSH;
  static constexpr int kBiases = HID * (1 + NH) + 16;
  static constexpr int kBiasOff = kFrags * 256;                  // words, inside the LDS image
  static constexpr int kImageBytes = (kBiasOff + kBiases) * 4;
  // offset (values) of layer l's weights inside the decoder's block
  static __host__ __device__ constexpr int layer_off(int l) {
    return l == 0 ? 0 : HID * (S::F + 1) + (l - 1) * HID * (HID + 1);
  }

  // Lane's 8 weights of fragment f, straight from the decoder's parameter block
  // p: one 16-byte load for layer 0 (units 32s + 8g ..), two 8-byte loads for
  // the others (the order the previous layer's accumulators leave its outputs
  // in).  The block is only 2-byte aligned in general (an odd output width), which
  // these loads allow.  Rows past the output width and units past the features
  // read weight 0 of the block and become zero.
  struct __attribute__((packed, aligned(2))) Piece16 { u32x4 v; };
  struct __attribute__((packed, aligned(2))) Piece8 { u32x2 v; };
  static __device__ __forceinline__ half8 load_slice(const uint16_t *p, int out_dim, int f,
                                                     int lane) {
    const int g = lane >> 4, n = lane & 15;
    if (f < kHidden0) {
      const int row = 16 * (f / S::KS0) + n, unit = 32 * (f % S::KS0) + 8 * g;
      const bool in = S::F % 32 == 0 || unit < S::F;
      const u32x4 v = ((const Piece16 *)(p + (in ? row * S::F + unit : 0)))->v;
      return as_half8(in ? v : u32x4{0u, 0u, 0u, 0u});
    }
    int row, s, off;
    bool in = true;
    if (f < kOut0) {
      const int q = f - kHidden0, layer = q / (S::MB * S::KSH), r = q % (S::MB * S::KSH);
      row = 16 * (r / S::KSH) + n;
      s = r % S::KSH;
      off = layer_off(1 + layer);
    } else {
      row = n;
      s = f - kOut0;
      off = layer_off(1 + NH);
      in = n < out_dim;
    }
    const uint16_t *src = p + (in ? off + row * HID + 32 * s + 4 * g : 0);
    const u32x2 lo = ((const Piece8 *)src)->v, hi = ((const Piece8 *)(src + 16))->v;
    return as_half8(in ? u32x4{lo[0], lo[1], hi[0], hi[1]} : u32x4{0u, 0u, 0u, 0u});
  }

  // Bias i of the image; the output layer's are scaled by -log2(e), so that
  // the sigmoid's exponent is one multiply-add, and zero past its width.
  static __device__ __forceinline__ float load_bias(const uint16_t *p, int out_dim, int i) {
    const bool out = i >= HID * (1 + NH);
    const int l = out ? 1 + NH : i / HID, row = out ? i - HID * (1 + NH) : i % HID;
    const bool in = !out || row < out_dim;
    const int dout = out ? out_dim : HID, din = l == 0 ? S::F : HID;
    const uint16_t hb = p[in ? layer_off(l) + dout * din + row : 0];
    const float v = (float)__builtin_bit_cast(_Float16, hb);
    return !in ? 0.f : out ? v * -kLog2e : v;
  }
};

// A decoder read from its LDS image.
template <int NL, int CH, int PE, int HID, int NH>
struct LdsNet : Net<NL, CH, PE, HID, NH> {
  using N = Net<NL, CH, PE, HID, NH>;
  const uint32_t *lds;
  __device__ __forceinline__ half8 weight(int f) const {
    return as_half8(*(const u32x4 *)(lds + (size_t)f * 256 + lane_id() * 4));
  }
  __device__ __forceinline__ const float *biases() const {
    return (const float *)lds + N::kBiasOff;
  }
};

// Bytes of the LDS cache of decoders below.
constexpr int kCacheBytes = 150 * 1024;

// A decoder whose weights this wave holds in registers and whose biases lie in
// LDS.
template <int NL, int CH, int PE, int HID, int NH>
struct RegNet : Net<NL, CH, PE, HID, NH> {
  using N = Net<NL, CH, PE, HID, NH>;
  half8 w[N::kFrags];
  float *lds;  // the wave's own region, N::kBiases floats
  const float *held;  // biases of the decoder in w: there, or in a cache slot
  __device__ __forceinline__ half8 weight(int f) const { return w[f]; }
  __device__ __forceinline__ const float *biases() const { return held; }
  // every fragment has arrived when this returns: a load left pending into the
  // caller's loop would be waited for on the path that loads nothing
  __device__ __forceinline__ void arrived() {
#pragma unroll
    for (int f = 0; f < N::kFrags; ++f) {
      u32x4 v = __builtin_bit_cast(u32x4, w[f]);
      asm volatile("" : "+v"(v));
      w[f] = as_half8(v);
    }
  }
  // Loads decoder `dec`: every load is issued before any is used.
  __device__ __forceinline__ void load(const DecodeArgs &a, uint32_t dec) {
    const uint16_t *p = a.params + (size_t)dec * (size_t)a.dec_stride;
    const int lane = (int)lane_id();
    constexpr int kPer = (N::kBiases + kWave - 1) / kWave;
    float b[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int k = i * kWave + lane;
      b[i] = N::load_bias(p, a.out_dim, k < N::kBiases ? k : 0);
    }
#pragma unroll
    for (int f = 0; f < N::kFrags; ++f) w[f] = N::load_slice(p, a.out_dim, f, lane);
    arrived();
    // the wave's earlier reads of the region come before these writes, and its
    // later ones after: a wave's LDS operations execute in order
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int k = i * kWave + lane;
      if (k < N::kBiases) lds[k] = b[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    held = lds;
  }

  // A workgroup's LDS cache of decoders (stream mode): kSlots images, decoder d
  // in slot d % kSlots, filled once by the first wave that misses there and
  // never replaced, so a filled slot is read without a lock and no wave waits
  // for another.  Of decoders that share a slot, the one that a wave came to first
  // is read from LDS and the others from memory for the whole call.  A tag is
  // kEmpty, kFilling or the decoder + 1.
  static constexpr uint32_t kSlots = (uint32_t)(kCacheBytes / N::kImageBytes);
  static constexpr uint32_t kEmpty = 0u, kFilling = 0xFFFFFFFFu;
  __device__ __forceinline__ void load_cached(const DecodeArgs &a, uint32_t dec, uint32_t *tags,
                                              uint32_t *images) {
    const int lane = (int)lane_id();
    const uint32_t slot = dec % kSlots;
    uint32_t *image = images + (size_t)slot * (N::kImageBytes / 4);
    const uint32_t tag = __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(&tags[slot], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
    if (tag == dec + 1) {
#pragma unroll
      for (int f = 0; f < N::kFrags; ++f)
        w[f] = as_half8(*(const u32x4 *)(image + f * 256 + lane * 4));
      arrived();
      held = (const float *)image + N::kBiasOff;
      return;
    }
    load(a, dec);
    if (tag != kEmpty) return;
    uint32_t was = kFilling;
    if (lane == 0) was = atomicCAS(&tags[slot], kEmpty, kFilling);
    if (__builtin_amdgcn_readfirstlane(was) != kEmpty) return;
#pragma unroll
    for (int f = 0; f < N::kFrags; ++f)
      *(u32x4 *)(image + f * 256 + lane * 4) = __builtin_bit_cast(u32x4, w[f]);
    for (int k = lane; k < N::kBiases; k += kWave) ((float *)image)[N::kBiasOff + k] = lds[k];
    if (lane == 0)
      __hip_atomic_store(&tags[slot], dec + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
};

// A decoder read straight from its parameter block, fragment by fragment
// (stream mode of 128-wide decoders), biases in the wave's own LDS region.
template <int NL, int CH, int PE, int HID, int NH>
struct DirectNet : Net<NL, CH, PE, HID, NH> {
  using N = Net<NL, CH, PE, HID, NH>;
  const uint16_t *p;
  int out_dim;
  float *lds;
  __device__ __forceinline__ half8 weight(int f) const {
    return N::load_slice(p, out_dim, f, (int)lane_id());
  }
  __device__ __forceinline__ const float *biases() const { return lds; }
  __device__ __forceinline__ void open(const DecodeArgs &a, uint32_t dec) {
    p = a.params + (size_t)dec * (size_t)a.dec_stride;
    out_dim = a.out_dim;
    for (int i = (int)lane_id(); i < N::kBiases; i += kWave) lds[i] = N::load_bias(p, out_dim, i);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
};

// Copies decoder `dec` into the LDS image; all threads of the workgroup take
// part and the caller brackets it with barriers.  A thread issues the loads of
// kStageSlices lane-slices back to back.
constexpr int kStageSlices = 4;

template <typename N, int THREADS>
__device__ void stage_decoder(const DecodeArgs &a, uint32_t dec, uint32_t *lds) {
  const uint16_t *p = a.params + (size_t)dec * (size_t)a.dec_stride;
  constexpr int kSlices = N::kFrags * kWave;
  for (int base = threadIdx.x; base < kSlices; base += kStageSlices * THREADS) {
    half8 v[kStageSlices];
#pragma unroll
    for (int i = 0; i < kStageSlices; ++i) {
      const int lf = base + i * THREADS;
      v[i] = N::load_slice(p, a.out_dim, (lf < kSlices ? lf : base) / kWave, lf % kWave);
    }
#pragma unroll
    for (int i = 0; i < kStageSlices; ++i) {
      const int lf = base + i * THREADS;
      if (lf < kSlices) *(half8 *)(lds + (size_t)lf * 4) = v[i];
    }
  }
  float *bias = (float *)lds + N::kBiasOff;
  for (int i = threadIdx.x; i < N::kBiases; i += THREADS) bias[i] = N::load_bias(p, a.out_dim, i);
}

// Positional encoding of the query's texture coordinate, PE / 4 octaves k:
// sin(2^k pi u), cos(2^k pi u), sin(2^k pi v), cos(2^k pi v), appended after
// the latent features as fp16 pairs (sin, cos).  v_sin_f32 / v_cos_f32 take
// the angle in turns: 2^k pi u is 2^(k-1) u turns, reduced to [0, 1) first
// (exact in fp32) so any finite coordinate stays inside the instructions'
// input range.
template <int PE>
__device__ __forceinline__ void pos_encoding(float u, float v, uint32_t *xo) {
#pragma unroll
  for (int k = 0; k < PE / 4; ++k) {
    const float scale = k == 0 ? 0.5f : (float)(1 << (k - 1));
    const float tu = __builtin_amdgcn_fractf(u * scale), tv = __builtin_amdgcn_fractf(v * scale);
    xo[2 * k] = pack_half2(__builtin_amdgcn_sinf(tu), __builtin_amdgcn_cosf(tu));
    xo[2 * k + 1] = pack_half2(__builtin_amdgcn_sinf(tv), __builtin_amdgcn_cosf(tv));
  }
}

// -------------------------------------------------------------------- gather

struct Query {
  uint32_t q;      // query index (only meaningful when valid)
  bool valid;
  uint32_t tex;
  float u, v, mip;
};

// The 2x2 texels of one level around a query and its position between them.
// fetch_level clamps the lower tap to [0, res - 2] and the weight to [0, 1]:
// for res >= 2 this is exactly bilinear filtering with both taps clamped to
// the edge, and it puts the right-hand tap 2*CH bytes after the left one (an
// immediate offset) and the lower row res*CH values further on.  Any finite
// or NaN coordinate keeps every tap inside the level.
template <int CH>
struct LevelTaps {
  static constexpr int NV = CH / 8;  // 16-byte vectors per texel
  u32x4 t00[NV], t10[NV], t01[NV], t11[NV];
  float fx, fy;
};

template <int CH>
__device__ __forceinline__ void fetch_level(const uint16_t *tex, uint32_t level_off, int res,
                                            float resf, float u, float v, LevelTaps<CH> &L) {
  const float x = __builtin_fmaf(u, resf, -0.5f), y = __builtin_fmaf(v, resf, -0.5f);
  const float hi = resf - 2.f;
  // med3 clamps (a NaN coordinate converts to index 0 below)
  const float x0 = __builtin_amdgcn_fmed3f(__builtin_floorf(x), 0.f, hi);
  const float y0 = __builtin_amdgcn_fmed3f(__builtin_floorf(y), 0.f, hi);
  L.fx = __builtin_amdgcn_fmed3f(x - x0, 0.f, 1.f);
  L.fy = __builtin_amdgcn_fmed3f(y - y0, 0.f, 1.f);
  const uint32_t idx = level_off + ((uint32_t)y0 * (uint32_t)res + (uint32_t)x0) * CH;
  const u32x4 *r0 = (const u32x4 *)(tex + idx);
  const u32x4 *r1 = (const u32x4 *)(tex + idx + (uint32_t)res * CH);
#pragma unroll
  for (int i = 0; i < LevelTaps<CH>::NV; ++i) {
    L.t00[i] = r0[i];
    L.t10[i] = r0[LevelTaps<CH>::NV + i];
    L.t01[i] = r1[i];
    L.t11[i] = r1[LevelTaps<CH>::NV + i];
  }
}

// Bilinear weights applied in packed fp16: each operation handles a channel
// pair, the four weights are rounded to fp16 and every product and sum is an
// fp16 operation (one v_pk_mul_f16 and three v_pk_fma_f16 per pair), half the
// instructions of an fp32 interpolation; its rounding stays well inside the
// decode tolerance.  Writes CH / 2 packed pairs, channel order.
__device__ __forceinline__ half2v as_h2(uint32_t v) { return __builtin_bit_cast(half2v, v); }

template <int CH>
__device__ __forceinline__ void interp_level_h2(const LevelTaps<CH> &L, uint32_t *xo) {
  const float gx = 1.f - L.fx, gy = 1.f - L.fy;
  const float2v w0 = {gx * gy, L.fx * gy}, w1 = {gx * L.fy, L.fx * L.fy};
  const half2v h0 = __builtin_convertvector(w0, half2v), h1 = __builtin_convertvector(w1, half2v);
  const half2v w00 = {h0[0], h0[0]}, w10 = {h0[1], h0[1]};
  const half2v w01 = {h1[0], h1[0]}, w11 = {h1[1], h1[1]};
#pragma unroll
  for (int i = 0; i < LevelTaps<CH>::NV; ++i) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      half2v r = as_h2(L.t00[i][e]) * w00;
      r = __builtin_elementwise_fma(as_h2(L.t10[i][e]), w10, r);
      r = __builtin_elementwise_fma(as_h2(L.t01[i][e]), w01, r);
      r = __builtin_elementwise_fma(as_h2(L.t11[i][e]), w11, r);
      xo[4 * i + e] = __builtin_bit_cast(uint32_t, r);
    }
  }
}

// v[k] for a per-lane level index k < NL, as a chain of selects (no scratch).
template <int NL, typename T>
__device__ __forceinline__ T pick(const T (&v)[NTC_MAX_LEVELS], int k) {
  T r = v[0];
#pragma unroll
  for (int i = 1; i < NL; ++i) r = k == i ? v[i] : r;
  return r;
}

// Feature vector of the lane's query, packed as fp16 pairs: x[c/2] holds
// features c and c+1; slot l occupies features [l*CH, (l+1)*CH).
template <int NL, int CH, int PE, bool MIP>
__device__ __forceinline__ void gather(const DecodeArgs &a, const Query &qq,
                                       uint32_t (&x)[(NL * CH + PE) / 2]) {
  if constexpr (PE > 0) pos_encoding<PE>(qq.u, qq.v, x + NL * CH / 2);
  const uint16_t *tex = a.latents + (size_t)qq.tex * (size_t)a.tex_stride;
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    if (!MIP) {
      LevelTaps<CH> L;
      fetch_level<CH>(tex, a.level_off[l], a.res[l], a.resf[l], qq.u, qq.v, L);
      interp_level_h2<CH>(L, x + l * CH / 2);
    } else {
      // Each level is interpolated in packed fp16 like the plain path, and the
      // blend f0 + t (f1 - f0) is one packed subtract and one packed fma per
      // pair (max-abs error of the decoded channels 9.7e-4 against 7.1e-4 for
      // an fp32 interpolation, 4 % less decode time on Wide + trilinear).  The
      // second level is fetched only when some lane of the wave blends: the
      // coarsest slot never does (its level of detail is always NL - 1).
      const float m = __builtin_fminf(__builtin_fmaxf(qq.mip, 0.f), (float)(NL - 1));
      const float lod = __builtin_fmaxf((float)l, m);
      const int k0 = (int)__builtin_floorf(lod);
      const int k1 = min(k0 + 1, NL - 1);
      const float t = lod - (float)k0;
      LevelTaps<CH> L0;
      fetch_level<CH>(tex, pick<NL>(a.level_off, k0), pick<NL>(a.res, k0), pick<NL>(a.resf, k0),
                      qq.u, qq.v, L0);
      interp_level_h2<CH>(L0, x + l * CH / 2);
      if (__builtin_amdgcn_ballot_w64(t != 0.f)) {
        LevelTaps<CH> L1;
        fetch_level<CH>(tex, pick<NL>(a.level_off, k1), pick<NL>(a.res, k1), pick<NL>(a.resf, k1),
                        qq.u, qq.v, L1);
        uint32_t f1[CH / 2];
        interp_level_h2<CH>(L1, f1);
        const _Float16 th = (_Float16)t;
        const half2v t2 = {th, th};
#pragma unroll
        for (int c = 0; c < CH / 2; ++c) {
          const half2v a0 = as_h2(x[l * CH / 2 + c]);
          x[l * CH / 2 + c] =
              __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(t2, as_h2(f1[c]) - a0, a0));
        }
      }
    }
  }
}

// Taps of all levels of one query, for the pipelined path without mip.
template <int NL, int CH>
struct TileTaps {
  LevelTaps<CH> lv[NL];
};

template <int NL, int CH>
__device__ __forceinline__ void fetch_taps(const DecodeArgs &a, const Query &qq,
                                           TileTaps<NL, CH> &T) {
  const uint16_t *tex = a.latents + (size_t)qq.tex * (size_t)a.tex_stride;
#pragma unroll
  for (int l = 0; l < NL; ++l)
    fetch_level<CH>(tex, a.level_off[l], a.res[l], a.resf[l], qq.u, qq.v, T.lv[l]);
}

template <int NL, int CH, int PE>
__device__ __forceinline__ void interp_taps(const TileTaps<NL, CH> &T,
                                            uint32_t (&x)[(NL * CH + PE) / 2]) {
#pragma unroll
  for (int l = 0; l < NL; ++l) interp_level_h2<CH>(T.lv[l], x + l * CH / 2);
}

// B operands of layer 0 from the features of the lane's own query (lane =
// query slot; x[c/2] holds features c, c+1): a 4x4 transpose of (16-lane row,
// 8-feature group) blocks per K-step, one v_permlane32_swap stage and one
// v_permlane16_swap stage.  Afterwards xb[j][s] holds, in lane (g, n),
// features 32s + 8g .. +7 of query 16j + n.
template <int KS0, int XW>
__device__ __forceinline__ void to_b16(const uint32_t (&x)[XW], half8 (&xb)[4][KS0]) {
#pragma unroll
  for (int s = 0; s < KS0; ++s) {
    uint32_t e[4][4];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int w = 16 * s + 4 * g + v;
        e[g][v] = w < XW ? x[w] : 0u;
      }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const auto a = __builtin_amdgcn_permlane32_swap(e[0][v], e[2][v], false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(e[1][v], e[3][v], false, false);
      e[0][v] = a[0]; e[2][v] = a[1];
      e[1][v] = b[0]; e[3][v] = b[1];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const auto a = __builtin_amdgcn_permlane16_swap(e[0][v], e[1][v], false, false);
      const auto b = __builtin_amdgcn_permlane16_swap(e[2][v], e[3][v], false, false);
      e[0][v] = a[0]; e[1][v] = a[1];
      e[2][v] = b[0]; e[3][v] = b[1];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) xb[j][s] = as_half8(u32x4{e[j][0], e[j][1], e[j][2], e[j][3]});
  }
}

// fp16 pair (round to nearest even) with ReLU applied on the packed halves: a
// negative half has its sign bit set, so a signed 16-bit max with 0 zeroes it.
// Rounding commutes with ReLU, so this equals rounding ReLU(x).
__device__ __forceinline__ uint32_t relu_pack2(float a, float b) {
  const short2v h = __builtin_bit_cast(short2v, pack_half2(a, b));
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(h, short2v{0, 0}));
}

// fp16 pair with LeakyReLU max(x, slope * x) (0 < slope < 1) applied on the
// packed halves, after rounding.
__device__ __forceinline__ uint32_t leaky_pack2(float a, float b, uint32_t slope_h2) {
  const half2v h = __builtin_bit_cast(half2v, pack_half2(a, b));
  const half2v s = __builtin_bit_cast(half2v, slope_h2);
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(h, h * s));
}

// Hidden activation and fp16 of row blocks 2t (lo) and 2t+1 (hi): the next
// layer's B operand for K-step t.
template <bool LEAKY>
__device__ __forceinline__ half8 act_pack16(const floatx4 &lo, const floatx4 &hi,
                                            uint32_t slope_h2) {
  if constexpr (LEAKY) {
    return as_half8(u32x4{leaky_pack2(lo[0], lo[1], slope_h2), leaky_pack2(lo[2], lo[3], slope_h2),
                          leaky_pack2(hi[0], hi[1], slope_h2), leaky_pack2(hi[2], hi[3], slope_h2)});
  } else {
    return as_half8(u32x4{relu_pack2(lo[0], lo[1]), relu_pack2(lo[2], lo[3]),
                          relu_pack2(hi[0], hi[1]), relu_pack2(hi[2], hi[3])});
  }
}

// 1 / (1 + exp(-(z + b))) with nb = -b * log2(e).
__device__ __forceinline__ float sigmoid(float z, float nb) {
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(__builtin_fmaf(z, -kLog2e, nb)));
}

// Two row blocks (2t, 2t+1) of a layer on the four column blocks, activated and
// converted: the next layer's B operand for K-step t.  KS K-steps, fragments
// from f0, biases of the two blocks at b.
template <int KS, bool LEAKY, typename NET>
__device__ __forceinline__ void row_pair(const NET &net, int f0, const float *b,
                                         const half8 (&x)[4][KS], half8 (&o)[4],
                                         uint32_t slope_h2) {
  const uint32_t g = lane_id() >> 4;
  const floatx4 blo = *(const floatx4 *)(b + 4 * g), bhi = *(const floatx4 *)(b + 16 + 4 * g);
  floatx4 lo[4], hi[4];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const half8 wlo = net.weight(f0 + s), whi = net.weight(f0 + KS + s);
#pragma unroll
    for (int j = 0; j < 4; ++j) lo[j] = mfma16(wlo, x[j][s], s == 0 ? blo : lo[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j) hi[j] = mfma16(whi, x[j][s], s == 0 ? bhi : hi[j]);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) o[j] = act_pack16<LEAKY>(lo[j], hi[j], slope_h2);
}

// Runs a decoder on the tile's features (B operands); y[j] holds the output
// layer's accumulators of column block j, bias not yet added.  The output layer
// takes each K-step as the last hidden layer produces it, so that layer's
// outputs are never all live.
template <int NL, int CH, int PE, int HID, int NH, bool LEAKY, typename NET>
__device__ __forceinline__ void mlp(const NET &net,
                                    const half8 (&xb)[4][Shape<NL, CH, PE, HID>::KS0],
                                    floatx4 (&y)[4], uint32_t slope_h2) {
  using S = Shape<NL, CH, PE, HID>;
  using N = Net<NL, CH, PE, HID, NH>;
  static_assert(NH >= 1, "a hidden -> hidden layer feeds the output layer");
  const float *bias = net.biases();
  half8 h[4][S::KSH];
#pragma unroll
  for (int t = 0; t < S::KSH; ++t) {
    half8 o[4];
    row_pair<S::KS0, LEAKY>(net, 2 * t * S::KS0, bias + 32 * t, xb, o, slope_h2);
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j][t] = o[j];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) y[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int layer = 0; layer < NH; ++layer) {
    half8 m[4][S::KSH];
#pragma unroll
    for (int t = 0; t < S::KSH; ++t) {
      half8 o[4];
      row_pair<S::KSH, LEAKY>(net, N::kHidden0 + layer * S::MB * S::KSH + 2 * t * S::KSH,
                              bias + HID * (1 + layer) + 32 * t, h, o, slope_h2);
      if (layer == NH - 1) {
        const half8 w = net.weight(N::kOut0 + t);
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = mfma16(w, o[j], y[j]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) m[j][t] = o[j];
      }
    }
    if (layer < NH - 1)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int t = 0; t < S::KSH; ++t) h[j][t] = m[j][t];
  }
}

// Raw buffer resource over the output rows: a store whose byte offset lies past
// the range is dropped by the hardware, so masked lanes need no branch and
// every path issues the same number of stores.  The output is at most
// kMaxOutBytes, so the drop offset (and the few 16-byte steps added to it) is
// past the range and offset + 16 never wraps around 32 bits.
constexpr uint32_t kDropOffset = 0xFFFFFF00u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t out_resource(const DecodeArgs &a) {
  const uint32_t bytes = a.n * (uint32_t)a.out_dim * (a.out_f16 ? 2u : 4u);  // <= kMaxOutBytes
  return __builtin_amdgcn_make_buffer_rsrc(a.out, 0, (int)bytes, 0x00020000);
}

// How a query's rows reach memory: for an output width of 4 or 8, one fp32 (or
// fp16) run of the 4 rows each lane holds; for a width of 3 (RGB rows, the
// Sec. 4 setup) the lanes holding rows 0..3 store rows 0..2 (fp32: one 12-byte
// store; fp16: a 4-byte and a 2-byte store); for any other width, one store per
// row (kStoreEach up to 8 rows, kStoreEachWide up to 16).
enum StoreMode { kStoreF32x4 = 0, kStoreF16x4 = 1, kStoreEach = 2, kStoreF32x3 = 3,
                 kStoreF16x3 = 4, kStoreEachWide = 5 };

// Widths past 8 need the accumulator rows 8..15.
template <int STORE>
constexpr bool kWideRows = STORE == kStoreEachWide;

// Store instructions per tile; fixed for a mode, so the wait counts of the
// software pipeline do not depend on the data.
template <int STORE>
constexpr int kStoresPerTile =
    STORE == kStoreEachWide ? 16 : STORE == kStoreEach ? 8 : STORE == kStoreF16x3 ? 4 : 2;

// Cache policy of the output stores: non-temporal.  The decoded rows are
// written once and not read again by the kernel; streaming them past the L2
// keeps the L2 for the latent texels that neighbouring queries share (about
// 13 % less decode time on the 4K clustered frame than default stores).
constexpr int kOutPolicy = 2;  // nt

// Every store of a mode is always issued (rows past the width, and masked
// lanes, get the drop offset), so the number of stores never depends on the
// data or the width.
// Decoded values of one lane for the store: rows r0 .. r0+3 of one query.
// Output widths up to 8 use the rows of lane groups 0 and 1 only; the upper
// half-wave of y[0] / y[1] takes y[2] / y[3]'s lower half first, so every lane
// finishes 4 values of y01[0] (queries 16n, blocks 0 / 2) and 4 of y01[1]
// (blocks 1 / 3).
// Bit casts through by-value helpers: a __builtin_bit_cast applied directly to
// an element of an ext_vector inside an unrolled loop is folded to element 0 by
// this compiler.
__device__ __forceinline__ uint32_t f32_bits(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ float bits_f32(uint32_t u) { return __builtin_bit_cast(float, u); }

__device__ __forceinline__ void compact_out(floatx4 (&y)[4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const auto a = __builtin_amdgcn_permlane32_swap(f32_bits(y[0][r]), f32_bits(y[2][r]), false,
                                                    false);
    const auto b = __builtin_amdgcn_permlane32_swap(f32_bits(y[1][r]), f32_bits(y[3][r]), false,
                                                    false);
    y[0][r] = bits_f32(a[0]);
    y[1][r] = bits_f32(b[0]);
  }
}

// Store of rows r0 .. r0 + 3 of query q (of the output's first 16 rows) in the
// given mode; rows at or past out_dim, and queries that are not ok, are
// dropped.
template <int STORE>
__device__ __forceinline__ void store4(__amdgpu_buffer_rsrc_t out, int out_dim, uint32_t q,
                                       bool ok, int r0, const u32x4 &v, uint32_t out_f16) {
  if constexpr (STORE == kStoreF32x4) {
    const uint32_t off = ok && r0 < out_dim ? (q * (uint32_t)out_dim + (uint32_t)r0) * 4u
                                            : kDropOffset;
    __builtin_amdgcn_raw_buffer_store_b128(v, out, off, 0, kOutPolicy);
  } else if constexpr (STORE == kStoreF16x4) {
    const uint32_t off = ok && r0 < out_dim ? (q * (uint32_t)out_dim + (uint32_t)r0) * 2u
                                            : kDropOffset;
    const float4 f = __builtin_bit_cast(float4, v);
    const u32x2 h = {pack_half2(f.x, f.y), pack_half2(f.z, f.w)};
    __builtin_amdgcn_raw_buffer_store_b64(h, out, off, 0, kOutPolicy);
  } else if constexpr (STORE == kStoreF32x3) {
    const uint32_t off = ok && r0 == 0 ? q * 12u : kDropOffset;
    const u32x3 w = {v[0], v[1], v[2]};
    __builtin_amdgcn_raw_buffer_store_b96(w, out, off, 0, kOutPolicy);
  } else if constexpr (STORE == kStoreF16x3) {
    const float4 f = __builtin_bit_cast(float4, v);
    const bool even = (q & 1u) == 0;
    const uint32_t base = q * 6u;
    const bool st = ok && r0 == 0;
    const uint32_t off32 = st ? (even ? base : base + 2u) : kDropOffset;
    const uint32_t off16 = st ? (even ? base + 4u : base) : kDropOffset;
    const uint32_t pair = even ? pack_half2(f.x, f.y) : pack_half2(f.y, f.z);
    const _Float16 single = (_Float16)(even ? f.z : f.x);
    __builtin_amdgcn_raw_buffer_store_b32(pair, out, off32, 0, kOutPolicy);
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, single), out, off16, 0,
                                           kOutPolicy);
  } else {
    const uint32_t row = q * (uint32_t)out_dim;
    const uint32_t es = out_f16 ? 2u : 4u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int rr = r0 + i;
      const uint32_t off = ok && rr < out_dim ? (row + (uint32_t)rr) * es : kDropOffset;
      if (out_f16) {
        const _Float16 f = (_Float16)bits_f32(v[i]);
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, f), out, off, 0,
                                               kOutPolicy);
      } else {
        __builtin_amdgcn_raw_buffer_store_b32(v[i], out, off, 0, kOutPolicy);
      }
    }
  }
}

// Finished output of a tile: sigmoid applied, with the query index and
// validity of each stored row group.  Widths up to 8 (WIDE = false) hold two
// 4-row groups per lane (after compact_out), wider outputs four.
template <bool WIDE>
struct TileOut {
  static constexpr int G = WIDE ? 4 : 2;
  u32x4 v[G];
  uint32_t q[G];
  uint32_t ok;   // bit i: group i is valid
};

// Sigmoid of the output accumulators with the scaled output biases; q and ok
// of the lane's own query slot (lane = query slot) are redistributed to the
// lanes that store its rows.
template <bool WIDE>
__device__ __forceinline__ TileOut<WIDE> finish16(floatx4 (&y)[4], const float *out_bias,
                                                  uint32_t q, bool ok) {
  TileOut<WIDE> o;
  const uint32_t lane = lane_id(), g = lane >> 4;
  const uint32_t okw = ok ? 1u : 0u;
  o.ok = 0;
  if constexpr (!WIDE) {
    compact_out(y);
    const floatx4 b = *(const floatx4 *)(out_bias + 4 * (g & 1));
    // lane (g, n) stores query slots (g < 2 ? n : 32 + n) and (g < 2 ? 16 + n : 48 + n)
    const auto qs = __builtin_amdgcn_permlane16_swap(q, q, false, false);
    const auto oks = __builtin_amdgcn_permlane16_swap(okw, okw, false, false);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) o.v[i][r] = f32_bits(sigmoid(y[i][r], b[r]));
      o.q[i] = qs[i];
      o.ok |= (oks[i] & 1u) << i;
    }
  } else {
    const floatx4 b = *(const floatx4 *)(out_bias + 4 * g);
    // lane (g, n) stores rows 4g .. 4g+3 of query slot 16j + n of each block j:
    // a 4x4 transpose of (row, block) of the query index and its validity
    uint32_t tq[4] = {q, q, q, q}, tk[4] = {okw, okw, okw, okw};
    {
      auto a = __builtin_amdgcn_permlane32_swap(tq[0], tq[2], false, false);
      auto b2 = __builtin_amdgcn_permlane32_swap(tq[1], tq[3], false, false);
      tq[0] = a[0]; tq[2] = a[1]; tq[1] = b2[0]; tq[3] = b2[1];
      a = __builtin_amdgcn_permlane16_swap(tq[0], tq[1], false, false);
      b2 = __builtin_amdgcn_permlane16_swap(tq[2], tq[3], false, false);
      tq[0] = a[0]; tq[1] = a[1]; tq[2] = b2[0]; tq[3] = b2[1];
      a = __builtin_amdgcn_permlane32_swap(tk[0], tk[2], false, false);
      b2 = __builtin_amdgcn_permlane32_swap(tk[1], tk[3], false, false);
      tk[0] = a[0]; tk[2] = a[1]; tk[1] = b2[0]; tk[3] = b2[1];
      a = __builtin_amdgcn_permlane16_swap(tk[0], tk[1], false, false);
      b2 = __builtin_amdgcn_permlane16_swap(tk[2], tk[3], false, false);
      tk[0] = a[0]; tk[1] = a[1]; tk[2] = b2[0]; tk[3] = b2[1];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int r = 0; r < 4; ++r) o.v[j][r] = f32_bits(sigmoid(y[j][r], b[r]));
      o.q[j] = tq[j];
      o.ok |= (tk[j] & 1u) << j;
    }
  }
  return o;
}

template <int STORE, bool WIDE>
__device__ __forceinline__ void store_out16(__amdgpu_buffer_rsrc_t out, int out_dim,
                                            const TileOut<WIDE> &o, uint32_t out_f16) {
  const uint32_t g = lane_id() >> 4;
  const int r0 = WIDE ? 4 * (int)g : 4 * (int)(g & 1);
#pragma unroll
  for (int i = 0; i < TileOut<WIDE>::G; ++i)
    store4<STORE>(out, out_dim, o.q[i], (o.ok >> i) & 1u, r0, o.v[i], out_f16);
}

// Query data of a slot.  The loads are unconditional (a slot without a valid
// query reads query 0), so every wave issues the same loads on every path and
// the compiler's waits stay exact.  The texture id is checked by validate(),
// once the tile that owns the query is about to use it.
template <int NL, bool MIP>
__device__ __forceinline__ Query load_query(const DecodeArgs &a, uint32_t q, bool in_range) {
  Query r;
  r.q = q;
  r.valid = in_range && q < a.n;
  const uint32_t qs = r.valid ? q : 0u;
  r.tex = a.tex_id[qs];
  const float2 uv = ((const float2 *)a.uv)[qs];
  r.u = uv.x;
  r.v = uv.y;
  r.mip = MIP ? a.mip[qs] : 0.f;
  return r;
}

// Marks a query with an out-of-range texture invalid and points it at texture
// 0, so its (discarded) gather stays inside the latents.
__device__ __forceinline__ Query validate(const DecodeArgs &a, Query r) {
  r.valid = r.valid && r.tex < (uint32_t)a.n_textures;
  if (!r.valid) r.tex = 0;
  return r;
}

// ------------------------------------------------------------------- kernels

typedef const __attribute__((address_space(4))) uint32_t *const_u32p;

// Wave-uniform read of the bin offsets through the constant address space, so
// it becomes a scalar load that does not enter the vector-memory counter.
__device__ __forceinline__ uint32_t bin_off(const DecodeArgs &a, uint32_t i) {
  return ((const_u32p)a.bin_offset)[i];
}

// A group of up to WAVES consecutive tiles of one bin: tiles [t, t + n) of bin
// d, whose tiles end at be; r counts the groups of a weighted sequence.  n == 0
// marks the end of a workgroup's range.
struct Group {
  uint32_t t, n, d, be;
  uint32_t r = 0;
};

template <int WAVES>
__device__ __forceinline__ Group group_at(const DecodeArgs &a, uint32_t t, uint32_t d,
                                          uint32_t be, uint32_t D, uint32_t t_end) {
  while (t >= be && d + 1 < D) {  // next non-empty bin
    ++d;
    be = bin_off(a, d + 1) / kWave;
  }
  const uint32_t n =
      (t >= be || t >= t_end) ? 0u : min(min((uint32_t)WAVES, be - t), t_end - t);
  return Group{t, n, d, be};
}

template <int WAVES>
__device__ __forceinline__ Group next_group(const DecodeArgs &a, const Group &g, uint32_t D,
                                            uint32_t t_end) {
  return g.n ? group_at<WAVES>(a, g.t + g.n, g.d, g.be, D, t_end) : g;
}

// Weighted groups: after every kRounds groups of up to WAVES tiles, one of up
// to WAVES / 2 tiles, for the first half of the waves only, so that the first
// half takes kRounds + 1 tiles for every kRounds of the second.  Waves w and
// w + WAVES / 2 of a workgroup share a SIMD, which issues the older wave, w,
// first.  Used by the binned decode of 128-wide decoders (2.64 -> 2.58 ms on
// the 4-sample trilinear 4K frame); with 64-wide ones it gained nothing on the
// 4K clustered frame and cost 2-4 % with positional encoding.
constexpr uint32_t kRounds = 6;

template <int WAVES>
__device__ __forceinline__ Group wgroup_at(const DecodeArgs &a, uint32_t t, uint32_t d,
                                           uint32_t be, uint32_t D, uint32_t t_end, uint32_t r) {
  Group g = group_at<WAVES>(a, t, d, be, D, t_end);
  if (r == kRounds) g.n = min(g.n, (uint32_t)WAVES / 2);
  g.r = r;
  return g;
}

template <int WAVES>
__device__ __forceinline__ Group next_wgroup(const DecodeArgs &a, const Group &g, uint32_t D,
                                             uint32_t t_end) {
  return g.n ? wgroup_at<WAVES>(a, g.t + g.n, g.d, g.be, D, t_end, g.r == kRounds ? 0u : g.r + 1)
             : g;
}

// Last bin whose first slot is at or before `slot` (wave uniform, below the
// total): 64 probes a round, one load each, so one round up to 64 decoders and
// two up to 4096; bin_offset[0] = 0 keeps the first probe true.
__device__ __forceinline__ uint32_t bin_of_slot(const DecodeArgs &a, uint32_t D, uint32_t slot) {
  const uint32_t lane = lane_id();
  uint32_t lo = 0, span = D;  // the bin lies in [lo, lo + span)
  while (span > 1) {
    const uint32_t step = (span + kWave - 1) / kWave;
    const uint32_t at = lane * step;
    const bool le = at < span && a.bin_offset[lo + (at < span ? at : 0u)] <= slot;
    const uint32_t k = (uint32_t)__builtin_popcountll(ballot(le)) - 1;
    lo += k * step;
    span = min(step, span - k * step);
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// Waves per workgroup of every kernel of the MFMA engine.
constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kWave;

// Waves per SIMD that the registers of the binned decode must allow: two workgroups
// per CU, or one for 128-wide decoders.  At four some shapes spill (two hidden layers
// with LeakyReLU, positional encoding: up to 60 bytes a lane) and are still faster
// than at three, where none does (1080p, two hidden layers, LeakyReLU, RGB: 79.6 us
// against 82.9 with 2 x 8 channels, 84.6 against 87.0 with 2 x 16).
template <int HID>
constexpr int kBinnedWavesPerSimd = HID == 64 ? 4 : 2;

// Weights in registers: stream order, 64-wide hidden layers (at most 26 fragments).
template <int HID>
constexpr bool kRegWeights = HID == 64;

// Taps ahead.  Stream: the taps of the next tile are fetched before this tile's MLP
// where they and the weights leave it its registers: up to 64 registers of taps (2
// levels of 16 channels) and 18 fragments.  Otherwise a tile gathers when it starts:
// carrying 3 levels' taps (96 registers) beside the weights spilled, as did 64 and a
// positional encoding (1080p frame of 16 decoders, 4 octaves 136 us against 103
// gathered in place, 8 octaves 140 against 114; 2 x 8 channels with 8 octaves fit, 94
// against 98).
template <int NL, int CH, int PE, int HID, int NH, bool MIP>
constexpr bool kStreamTapsAhead =
    kRegWeights<HID> && !MIP && NL * CH <= (PE > 0 ? 16 : 32) &&
    Net<NL, CH, PE, HID, NH>::kFrags <= 18;
// Binned: fetched before this tile's stores for 128-wide decoders; with four waves a
// SIMD the other waves hide a gather at the tile's start (1080p one material, passes
// of 51.2 us against 52.9 fetched ahead; 3 levels, 70.9 against 86).
template <int HID, bool MIP>
constexpr bool kBinnedTapsAhead = !MIP && HID > 64;

// Binned decode with the weights in LDS: a workgroup walks a contiguous range of
// tiles, one a wave at a time inside one bin, restaging the decoder when the bin
// changes.  split: twice the tiles for the first workgroup dispatched to each CU
// (blockIdx < gridDim / 2) of two: the SIMDs issue the older waves first, so two with
// equal work finish a third apart and the second runs its last third on half the
// waves (4K frame of 2 x 16 channels with mip 214.9 -> 207.2 us, 1080p 70.0 -> 67.7).
template <int NL, int CH, int PE, int HID, int NH, bool MIP, int STORE, bool LEAKY>
__global__ void __launch_bounds__(kThreads, kBinnedWavesPerSimd<HID>)
decode_binned(const DecodeArgs a, uint32_t split) {
  using S = Shape<NL, CH, PE, HID>;
  using N = Net<NL, CH, PE, HID, NH>;
  constexpr bool WIDE = kWideRows<STORE>;
  constexpr bool AHEAD = kBinnedTapsAhead<HID, MIP>;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  const uint32_t lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t D = (uint32_t)a.n_decoders;
  const __amdgpu_buffer_rsrc_t out_rsrc = out_resource(a);
  const uint64_t slots = min((uint64_t)bin_off(a, D), a.perm_capacity);
  const uint32_t total_tiles = (uint32_t)(slots / kWave);
  uint32_t t, t_end;
  if (HID == 64 && split) {  // 128-wide: one workgroup a CU
    const uint32_t half = gridDim.x / 16, xcd = blockIdx.x % 8, j = blockIdx.x / 8;
    const uint64_t w0 = (uint64_t)xcd * half * 3 + (j < half ? 2 * j : half + j);
    const uint64_t w1 = w0 + (j < half ? 2 : 1), parts = (uint64_t)gridDim.x / 2 * 3;
    t = (uint32_t)(total_tiles * w0 / parts);
    t_end = (uint32_t)(total_tiles * w1 / parts);
  } else {
    const uint32_t per = (total_tiles + gridDim.x - 1) / gridDim.x;
    t = xcd_local_block(blockIdx.x, gridDim.x) * per;
    t_end = min(t + per, total_tiles);
  }
  if (t >= t_end) return;
  const uint32_t first = bin_of_slot(a, D, t * kWave);
  // Tiles go in (128-wide: weighted) groups of consecutive tiles of one bin, tile
  // t + w to wave w; every wave walks the same (uniform) sequence of groups.  A wave
  // without a tile in a group skips its MLP and stores but still takes part in
  // its staging and prefetches.
  auto next = [&](const Group &g) {
    return HID > 64 ? next_wgroup<kWaves>(a, g, D, t_end) : next_group<kWaves>(a, g, D, t_end);
  };
  Group g0 = group_at<kWaves>(a, t, first, bin_off(a, first + 1) / kWave, D, t_end);
  Group g1 = next(g0);
  Group g2 = next(g1);
  Group g3 = next(g2);
  struct Slot {
    uint32_t raw;
    bool has;
  };
  auto slot_query = [&](const Group &g) -> Slot {
    const bool has = w < g.n;
    return Slot{a.perm[has ? (g.t + w) * kWave + lane : 0u], has};
  };
  auto restage = [&](uint32_t d) {
    __syncthreads();  // every wave is done with the previous decoder
    stage_decoder<N, kThreads>(a, d, lds);
    __syncthreads();
  };
  LdsNet<NL, CH, PE, HID, NH> net;
  net.lds = lds;
  const Slot s0 = slot_query(g0);
  Query cur = validate(a, load_query<NL, MIP>(a, s0.raw, s0.has));  // tile 0
  restage(g0.d);
  uint32_t staged = g0.d;
  TileTaps<NL, CH> taps;
  if constexpr (AHEAD) fetch_taps<NL, CH>(a, cur, taps);
  __builtin_amdgcn_sched_barrier(0);
  const Slot s1 = slot_query(g1);
  Query q_next = load_query<NL, MIP>(a, s1.raw, s1.has);  // tile 1
  Slot p_next = slot_query(g2);                            // tile 2
  __builtin_amdgcn_sched_barrier(0);
  // As many stores as a loop iteration issues, all past the range (dropped):
  // the loop is entered with the same operations in flight, in the same
  // order, as at its back edge, so the waits at its top need not drain.
  // Distinct offsets keep them from being merged.
#pragma unroll
  for (uint32_t i = 0; i < kStoresPerTile<STORE>; ++i)
    __builtin_amdgcn_raw_buffer_store_b32(0u, out_rsrc, kDropOffset + 16u * i, 0, 0);
  auto tile = [&](const Query &q_in, const Slot &p_in, Query &q_out, Slot &p_out) {
    const bool busy = w < g0.n;  // this wave has a tile in the group
    TileOut<WIDE> o;
    if (busy) {
      uint32_t x[S::F / 2];
      if constexpr (!AHEAD) {
        gather<NL, CH, PE, MIP>(a, cur, x);
      } else {
        interp_taps<NL, CH, PE>(taps, x);
        if constexpr (PE > 0) pos_encoding<PE>(cur.u, cur.v, x + NL * CH / 2);
      }
      half8 xb[4][S::KS0];
      to_b16<S::KS0, S::F / 2>(x, xb);
      floatx4 y[4];
      mlp<NL, CH, PE, HID, NH, LEAKY>(net, xb, y, a.slope_h2);
      o = finish16<WIDE>(y, net.biases() + HID * (1 + NH), cur.q, cur.valid);
    }
    __builtin_amdgcn_sched_barrier(0);
    // The next group's decoder is staged here, between this tile's MLP and the
    // next tile's fetches, so no fetched data is live across the staging.
    if (g1.n && g1.d != staged) {
      restage(g1.d);
      staged = g1.d;
    }
    // next tile: taps, then the prefetches, then this tile's stores
    const Query nxt = validate(a, q_in);
    if constexpr (AHEAD) fetch_taps<NL, CH>(a, nxt, taps);
    __builtin_amdgcn_sched_barrier(0);
    q_out = load_query<NL, MIP>(a, p_in.raw, p_in.has);
    p_out = slot_query(g3);
    __builtin_amdgcn_sched_barrier(0);
    if (busy) store_out16<STORE, WIDE>(out_rsrc, a.out_dim, o, a.out_f16);
    cur = nxt;
    g0 = g1;
    g1 = g2;
    g2 = g3;
    g3 = next(g3);
  };
  Query q_b;
  Slot p_b;
  for (;;) {
    if (!g0.n) break;
    tile(q_next, p_next, q_b, p_b);
    if (!g0.n) break;
    tile(q_b, p_b, q_next, p_next);
  }
}

// ---------------------------------------------------------------- stream mode
//
// The paper's non-shared tensor decoder (Sec. 4.4): a wave pays one full MLP
// pass per decoder its tile holds.

// Decoder of a validated query, kNoDecoder for none.  The load is unconditional
// (validate() points an invalid query at texture 0).
constexpr uint32_t kNoDecoder = 0xFFFFFFFFu;
__device__ __forceinline__ uint32_t decoder_of(const DecodeArgs &a, const Query &q, uint32_t dd) {
  return q.valid && dd < (uint32_t)a.n_decoders ? dd : kNoDecoder;
}

// Stream decode with the weights in registers (64-wide decoders).  Every wave
// walks a contiguous run of tiles and keeps the last decoder it used: a tile
// takes the held decoder first, then loads each other one it needs, so a run
// over one material loads nothing.  The other loads come from an LDS cache of
// decoders where the workgroup has one (`cached`), else from the parameter
// blocks.  What bounds it is the latency of those loads and, on frames of one
// material, what bounds the binned decode.  1080p frame of 16 decoders: 192 us
// when every wave read each fragment of each pass through the caches, 129 with
// the held decoder, 88 with the LDS cache.
template <int NL, int CH, int PE, int HID, int NH, bool MIP, int STORE, bool LEAKY>
__global__ void __launch_bounds__(kThreads, 2) decode_stream_reg(const DecodeArgs a, uint32_t cached) {
  using S = Shape<NL, CH, PE, HID>;
  using N = Net<NL, CH, PE, HID, NH>;
  using R = RegNet<NL, CH, PE, HID, NH>;
  constexpr bool AHEAD = kStreamTapsAhead<NL, CH, PE, HID, NH, MIP>;
  constexpr bool WIDE = kWideRows<STORE>;
  __shared__ __attribute__((aligned(16))) float biases[kWaves][N::kBiases];
  __shared__ uint32_t tags[R::kSlots];
  extern __shared__ __attribute__((aligned(16))) uint32_t images[];  // cached: kSlots images
  const uint32_t lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const __amdgpu_buffer_rsrc_t out_rsrc = out_resource(a);
  const uint32_t n_tiles = (uint32_t)(((uint64_t)a.n + kWave - 1) / kWave);
  const uint32_t nw = blockDim.x / kWave;  // waves of this workgroup, at most kWaves
  if (threadIdx.x < R::kSlots) tags[threadIdx.x] = R::kEmpty;
  __syncthreads();
  const uint64_t waves = (uint64_t)gridDim.x * nw;
  const uint64_t me = (uint64_t)xcd_local_block(blockIdx.x, gridDim.x) * nw + w;
  const uint32_t t_beg = (uint32_t)(n_tiles * me / waves);
  const uint32_t t_end = (uint32_t)(n_tiles * (me + 1) / waves);
  if (t_beg >= t_end) return;
  auto query_of = [&](uint32_t t) { return load_query<NL, MIP>(a, t * kWave + lane, t < t_end); };
  R net;
  net.lds = biases[w];
  net.held = biases[w];
  uint32_t held = kNoDecoder;
  Query cur = query_of(t_beg);
  Query q_next = query_of(t_beg + 1);
  cur = validate(a, cur);
  uint32_t dd = a.tex_to_dec[cur.tex];
  TileTaps<NL, CH> taps;
  if constexpr (AHEAD) fetch_taps<NL, CH>(a, cur, taps);
  for (uint32_t t = t_beg; t < t_end; ++t) {
    uint32_t x[S::F / 2];
    if constexpr (AHEAD) {
      interp_taps<NL, CH, PE>(taps, x);
      if constexpr (PE > 0) pos_encoding<PE>(cur.u, cur.v, x + NL * CH / 2);
    } else {
      gather<NL, CH, PE, MIP>(a, cur, x);
    }
    const uint32_t dq = decoder_of(a, cur, dd);
    const Query nxt = validate(a, q_next);
    if constexpr (AHEAD) fetch_taps<NL, CH>(a, nxt, taps);
    dd = a.tex_to_dec[nxt.tex];
    q_next = query_of(t + 2);
    half8 xb[4][S::KS0];
    to_b16<S::KS0, S::F / 2>(x, xb);
    __builtin_amdgcn_sched_barrier(0);
    uint64_t todo = ballot(dq != kNoDecoder);
    while (todo) {
      uint64_t mine = ballot(dq == held) & todo;
      if (!mine) {
        held = read_lane(dq, (uint32_t)__builtin_ctzll(todo));
        mine = ballot(dq == held);
        if (cached) net.load_cached(a, held, tags, images);
        else net.load(a, held);
      }
      floatx4 y[4];
      mlp<NL, CH, PE, HID, NH, LEAKY>(net, xb, y, a.slope_h2);
      const TileOut<WIDE> o =
          finish16<WIDE>(y, net.biases() + HID * (1 + NH), cur.q, (mine >> lane) & 1);
      store_out16<STORE, WIDE>(out_rsrc, a.out_dim, o, a.out_f16);
      todo &= ~mine;
    }
    cur = nxt;
  }
}

// Stream decode of 128-wide decoders.  A workgroup takes groups of eight
// consecutive tiles, one per wave.  At every kStreamVoteEvery-th group the waves
// vote: when all of them hold one and the same decoder, it is staged once in
// LDS, and every wave reads it from there until a later vote stages another.
// Any other decoder a wave holds, the wave evaluates on its own, reading every
// MFMA A fragment straight from that decoder's parameter block, with no
// restaging and no barrier.  Restaging the union of a group's decoders in LDS
// would make every wave wait for every decoder of the group; per-wave reads
// alone are twice as slow as one staged copy when waves share a decoder.  1080p frame
// of 16 decoders: 48-128-128-128-8 1201 us (1506 with 32x32x16 MFMAs), 32-128-128-8
// 605 (662).  With two hidden layers the per-wave path spills 130-310 bytes a lane
// (210-330 before); it waits for its fragments from memory in any case.
constexpr uint32_t kStreamVoteEvery = 8;

template <int NL, int CH, int PE, int HID, int NH, bool MIP, int STORE, bool LEAKY>
__global__ void __launch_bounds__(kThreads, 1)
decode_stream_mixed(const DecodeArgs a, uint32_t image_bytes) {
  constexpr uint32_t kNone = kNoDecoder, kMixed = 0xFFFFFFFEu;
  using S = Shape<NL, CH, PE, HID>;
  using N = Net<NL, CH, PE, HID, NH>;
  constexpr bool WIDE = kWideRows<STORE>;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  __shared__ uint32_t wave_dec[2][kWaves];
  const uint32_t w = threadIdx.x / kWave, lane = lane_id();
  const __amdgpu_buffer_rsrc_t out_rsrc = out_resource(a);
  const uint32_t n_tiles = (uint32_t)(((uint64_t)a.n + kWave - 1) / kWave);
  const uint32_t n_groups = (n_tiles + kWaves - 1) / kWaves;
  const uint32_t per = (n_groups + gridDim.x - 1) / gridDim.x;
  const uint32_t blk = xcd_local_block(blockIdx.x, gridDim.x);
  const uint32_t g_begin = blk * per, g_end = min(g_begin + per, n_groups);
  LdsNet<NL, CH, PE, HID, NH> shared;
  shared.lds = lds;
  DirectNet<NL, CH, PE, HID, NH> own;
  own.lds = (float *)(lds + image_bytes / 4) + (size_t)w * N::kBiases;  // this wave's region
  uint32_t staged = kNone;  // the decoder in the shared image; the same in every wave
  int parity = 0;
  for (uint32_t g = g_begin; g < g_end; ++g) {
    const uint64_t q64 = ((uint64_t)g * kWaves + w) * kWave + lane;
    const uint32_t q = (uint32_t)q64;
    const Query qq = validate(a, load_query<NL, MIP>(a, q, q64 < a.n));
    const uint32_t dq = decoder_of(a, qq, a.tex_to_dec[qq.tex]);
    uint32_t x[S::F / 2];
    gather<NL, CH, PE, MIP>(a, qq, x);
    half8 xb[4][S::KS0];
    to_b16<S::KS0, S::F / 2>(x, xb);
    uint64_t todo = ballot(dq != kNone);
    // the wave's one decoder, kMixed for several, kNone for none
    if ((g - g_begin) % kStreamVoteEvery == 0) {
      const uint32_t first = todo ? read_lane(dq, (uint32_t)__builtin_ctzll(todo)) : kNone;
      const uint32_t mine_one = ballot(dq != kNone && dq != first) ? kMixed : first;
      if (lane == 0) wave_dec[parity][w] = mine_one;
      __syncthreads();  // also: every wave is done with its reads of the staged image
      uint32_t common = kNone;
      bool agree = true;
#pragma unroll
      for (int k = 0; k < kWaves; ++k) {
        const uint32_t v = wave_dec[parity][k];
        if (v == kNone) continue;
        if (v == kMixed || (common != kNone && v != common)) agree = false;
        common = v;
      }
      parity ^= 1;
      if (agree && common != kNone && common != staged) {
        // every wave of the group holds this one decoder: share one staged copy
        stage_decoder<N, kThreads>(a, common, lds);
        __syncthreads();
        staged = common;
      }
    }
    while (todo) {
      const uint32_t d = read_lane(dq, (uint32_t)__builtin_ctzll(todo));
      const bool mine = dq == d;
      floatx4 y[4];
      const float *ob;
      if (d == staged) {
        mlp<NL, CH, PE, HID, NH, LEAKY>(shared, xb, y, a.slope_h2);
        ob = shared.biases();
      } else {
        own.open(a, d);
        mlp<NL, CH, PE, HID, NH, LEAKY>(own, xb, y, a.slope_h2);
        ob = own.biases();
      }
      const TileOut<WIDE> o = finish16<WIDE>(y, ob + HID * (1 + NH), q, mine);
      store_out16<STORE, WIDE>(out_rsrc, a.out_dim, o, a.out_f16);
      todo &= ~ballot(mine);
    }
  }
}

// ------------------------------------------------- non-shared FMA decode
//
// The paper's Non-Shared FMA comparison (Sec. 4.4): every lane evaluates the
// decoder of its own query with vector instructions, so lanes that use
// different decoders share one instruction stream and differ only in the
// addresses their weights come from; the cost does not grow with the number of
// decoders in a wave, unlike the tensor path's one pass per decoder.  Products
// are v_dot2c_f32_f16 (two fp16 products added to an fp32 accumulator), with
// the tensor path's fp16 features and fp16-rounded activations, so both engines
// compute the same function within rounding.
//
// One thread per query, stream order.  Row j of W_i is read by the lane as
// din / 8 16-byte loads from the lane's decoder block (L1/L2-cached).  A layer
// takes its input from registers and writes its output, as fp16 pairs, to the
// thread's own LDS column (word i at i * kBlock + thread): the row loop is a
// runtime loop, and registers cannot be indexed at run time.

__device__ __forceinline__ float dot2(uint32_t w, uint32_t h, float c) {
  return __builtin_amdgcn_fdot2(as_h2(w), as_h2(h), c, false);
}

// fp16 pair of two fp32 values.
__device__ __forceinline__ float2 unpack_half2(uint32_t v) {
  const half2v h = as_h2(v);
  return float2{(float)h[0], (float)h[1]};
}

// Layer din -> dout (dout even) with its input h (fp16 pairs) in registers.
// Hidden layers (OUT = false) write the activated outputs as fp16 pairs, word
// j / 2 of the thread's LDS column; the output layer (OUT = true) writes the
// sigmoid of each output as a float, word j.
template <int DIN, bool OUT>
__device__ __forceinline__ void fma_layer(const uint16_t *W, int dout, const uint32_t (&h)[DIN / 2],
                                          uint32_t *col, bool leaky, uint32_t slope_h2) {
  const uint16_t *b = W + (size_t)dout * DIN;
#pragma unroll 2
  for (int j = 0; j < dout; j += 2) {
    const float2 bj = unpack_half2(*(const uint32_t *)(b + j));
    float acc0 = bj.x, acc1 = bj.y;
    const u32x4 *r0 = (const u32x4 *)(W + (size_t)j * DIN);
    const u32x4 *r1 = (const u32x4 *)(W + (size_t)(j + 1) * DIN);
#pragma unroll
    for (int k = 0; k < DIN / 8; ++k) {
      const u32x4 w0 = r0[k], w1 = r1[k];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc0 = dot2(w0[e], h[4 * k + e], acc0);
        acc1 = dot2(w1[e], h[4 * k + e], acc1);
      }
    }
    if constexpr (OUT) {
      col[j * kBlock] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(acc0 * -kLog2e)));
      col[(j + 1) * kBlock] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(acc1 * -kLog2e)));
    } else {
      col[(j / 2) * kBlock] = leaky ? leaky_pack2(acc0, acc1, slope_h2) : relu_pack2(acc0, acc1);
    }
  }
}

// Words of a thread's LDS column: the widest hidden layer as fp16 pairs, or the
// output row as floats.
template <int HID>
constexpr int kFmaColumn = HID / 2 > 16 ? HID / 2 : 16;

template <int NL, int CH, int PE, int HID, bool MIP>
__global__ void __launch_bounds__(kBlock, 2) decode_fma(const DecodeArgs a) {
  using S = Shape<NL, CH, PE, HID>;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  uint32_t *col = lds + threadIdx.x;  // this thread's activations, stride kBlock
  const uint64_t q64 = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (q64 >= a.n) return;
  const uint32_t q = (uint32_t)q64;
  const Query qq = validate(a, load_query<NL, MIP>(a, q, true));
  if (!qq.valid) return;
  const uint32_t d = a.tex_to_dec[qq.tex];
  if (d >= (uint32_t)a.n_decoders) return;
  const uint16_t *p = a.params + (size_t)d * (size_t)a.dec_stride;
  const bool leaky = a.leaky != 0;
  {  // layer 0: F -> HID
    uint32_t x[S::F / 2];
    gather<NL, CH, PE, MIP>(a, qq, x);
    fma_layer<S::F, false>(p, HID, x, col, leaky, a.slope_h2);
    p += (size_t)HID * (S::F + 1);
  }
  // hidden -> hidden, then the output layer (8 or 16 wide, sigmoid)
  for (int l = 0; l <= a.n_hidden; ++l) {
    uint32_t h[HID / 2];
#pragma unroll
    for (int i = 0; i < HID / 2; ++i) h[i] = col[i * kBlock];
    if (l < a.n_hidden) {
      fma_layer<HID, false>(p, HID, h, col, leaky, a.slope_h2);
      p += (size_t)HID * (HID + 1);
    } else {
      fma_layer<HID, true>(p, a.out_dim, h, col, leaky, a.slope_h2);
    }
  }
  const int out_dim = a.out_dim;
  float y[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) y[c] = c < out_dim ? __builtin_bit_cast(float, col[c * kBlock]) : 0.f;
  if (a.out_f16) {
    u32x2 *o = (u32x2 *)((uint16_t *)a.out + (size_t)q * out_dim);
#pragma unroll
    for (int c = 0; c < 16; c += 4)
      if (c < out_dim) o[c / 4] = u32x2{pack_half2(y[c], y[c + 1]), pack_half2(y[c + 2], y[c + 3])};
  } else {
    floatx4 *o = (floatx4 *)((float *)a.out + (size_t)q * out_dim);
#pragma unroll
    for (int c = 0; c < 16; c += 4)
      if (c < out_dim) o[c / 4] = floatx4{y[c], y[c + 1], y[c + 2], y[c + 3]};
  }
}

template <int NL, int CH, int PE, int HID, bool MIP>
int launch_fma(const DecodeArgs &a, hipStream_t stream) {
  const void *fn = (const void *)decode_fma<NL, CH, PE, HID, MIP>;
  const size_t lds = (size_t)kFmaColumn<HID> * kBlock * sizeof(uint32_t);
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return NTC_ERR_HIP;
  const uint64_t blocks = ((uint64_t)a.n + kBlock - 1) / kBlock;
  hipLaunchKernelGGL((decode_fma<NL, CH, PE, HID, MIP>), dim3((unsigned)blocks), dim3(kBlock), lds,
                     stream, a);
  return hip_status(hipGetLastError());
}

// ------------------------------------- non-shared FMA decode, LDS weight cache
//
// The same per-lane computation with the weights read from LDS: one workgroup
// of kFmaLdsThreads threads per CU walks tiles of that many consecutive
// queries and keeps up to `slots` whole decoders in an LDS cache.  For each
// tile it looks up every query's decoder, stages the missing ones into slots
// no pending query of the tile uses (one cooperative copy), and every lane
// whose decoder is cached evaluates its own query with v_dot2c_f32_f16 on rows
// read from its decoder's slot; a tile with more distinct decoders than slots
// takes several passes.  Lanes of one wave that use different decoders read
// different slots in one instruction.  Hidden width 64: activations stay in
// registers (the row loops are unrolled).
constexpr int kFmaLdsThreads = 1024;
constexpr int kFmaLdsWaves = kFmaLdsThreads / kWave;
constexpr size_t kFmaLdsWeightBytes = 144 * 1024;  // the decoder cache
constexpr uint32_t kFmaMaxSlots = 16;
constexpr uint32_t kNoSlotDecoder = 0xFFFFFFFFu;

struct FmaCache {
  uint32_t slot_dec[kFmaMaxSlots];  // decoder held by each slot
  uint32_t used[kFmaMaxSlots];      // a pending query of this pass hit the slot
  uint32_t want[kFmaLdsWaves][kFmaMaxSlots];  // per wave: distinct missing decoders
  uint32_t n_want[kFmaLdsWaves];
  uint32_t stage_slot[kFmaMaxSlots], stage_dec[kFmaMaxSlots];
  uint32_t n_stage;
};

// Layer DIN -> 64 (activated, fp16 pairs) from a decoder's weights in LDS.
template <int DIN>
__device__ __forceinline__ void fma_hidden_lds(const uint16_t *W, const uint32_t (&h)[DIN / 2],
                                               uint32_t (&o)[32], bool leaky, uint32_t slope_h2) {
  const uint16_t *b = W + 64 * DIN;
#pragma unroll
  for (int j = 0; j < 64; j += 2) {
    const float2 bj = unpack_half2(*(const uint32_t *)(b + j));
    float acc0 = bj.x, acc1 = bj.y;
    const u32x4 *r0 = (const u32x4 *)(W + j * DIN);
    const u32x4 *r1 = (const u32x4 *)(W + (j + 1) * DIN);
#pragma unroll
    for (int k = 0; k < DIN / 8; ++k) {
      const u32x4 w0 = r0[k], w1 = r1[k];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc0 = dot2(w0[e], h[4 * k + e], acc0);
        acc1 = dot2(w1[e], h[4 * k + e], acc1);
      }
    }
    o[j / 2] = leaky ? leaky_pack2(acc0, acc1, slope_h2) : relu_pack2(acc0, acc1);
  }
}

// Output layer 64 -> dout (8 or 16), logistic sigmoid, from LDS.
__device__ __forceinline__ void fma_out_lds(const uint16_t *W, int dout, const uint32_t (&h)[32],
                                            float (&y)[16]) {
  const uint16_t *b = W + dout * 64;
#pragma unroll
  for (int j = 0; j < 16; j += 2) {
    if (j < dout) {
      const float2 bj = unpack_half2(*(const uint32_t *)(b + j));
      float acc0 = bj.x, acc1 = bj.y;
      const u32x4 *r0 = (const u32x4 *)(W + j * 64);
      const u32x4 *r1 = (const u32x4 *)(W + (j + 1) * 64);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const u32x4 w0 = r0[k], w1 = r1[k];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc0 = dot2(w0[e], h[4 * k + e], acc0);
          acc1 = dot2(w1[e], h[4 * k + e], acc1);
        }
      }
      y[j] = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(acc0 * -kLog2e));
      y[j + 1] = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(acc1 * -kLog2e));
    } else {
      y[j] = y[j + 1] = 0.f;
    }
  }
}

template <int NL, int CH, int PE, bool MIP>
__global__ void __launch_bounds__(kFmaLdsThreads)
decode_fma_lds(const DecodeArgs a, uint32_t slots, uint32_t n_tiles) {
  using S = Shape<NL, CH, PE, 64>;
  extern __shared__ __attribute__((aligned(16))) uint16_t wcache[];
  __shared__ FmaCache c;
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const uint32_t stride = (uint32_t)a.dec_stride;  // halves, a multiple of 8
  const uint32_t D = (uint32_t)a.n_decoders;
  const bool leaky = a.leaky != 0;
  if (tid < kFmaMaxSlots) {
    c.slot_dec[tid] = kNoSlotDecoder;
    c.used[tid] = 0;
  }
  for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const uint64_t q64 = (uint64_t)tile * kFmaLdsThreads + tid;
    const uint32_t q = (uint32_t)q64;
    const Query qq = validate(a, load_query<NL, MIP>(a, q, q64 < a.n));
    uint32_t d = qq.valid ? a.tex_to_dec[qq.tex] : kNoSlotDecoder;
    if (d >= D) d = kNoSlotDecoder;
    bool pending = d != kNoSlotDecoder;
    uint32_t x[S::F / 2];
    gather<NL, CH, PE, MIP>(a, qq, x);  // an invalid query gathers texture 0, unused
    while (__syncthreads_or(pending)) {
      // look the decoder up; mark the slots this pass reads; list the misses
      int slot = -1;
      if (pending)
        for (uint32_t k = 0; k < slots; ++k)
          if (c.slot_dec[k] == d) slot = (int)k;
      if (pending && slot >= 0) c.used[slot] = 1;
      const bool miss = pending && slot < 0;
      uint64_t todo = ballot(miss);
      uint32_t nw = 0;
      while (todo) {
        const uint32_t dl = read_lane(d, (uint32_t)__builtin_ctzll(todo));
        todo &= ~ballot(d == dl);
        if (lane == 0 && nw < kFmaMaxSlots) c.want[w][nw] = dl;
        ++nw;
      }
      if (lane == 0) c.n_want[w] = nw < kFmaMaxSlots ? nw : kFmaMaxSlots;
      __syncthreads();
      // one thread plans: distinct wanted decoders into slots no pending query hit
      if (tid == 0) {
        uint32_t ns = 0, next = 0;
        bool full = false;
        for (int wv = 0; wv < kFmaLdsWaves && !full; ++wv)
          for (uint32_t i = 0; i < c.n_want[wv] && !full; ++i) {
            const uint32_t dl = c.want[wv][i];
            bool dup = false;
            for (uint32_t k = 0; k < ns; ++k) dup = dup || c.stage_dec[k] == dl;
            if (dup) continue;
            while (next < slots && c.used[next]) ++next;
            if (next == slots) {
              full = true;
              break;
            }
            c.stage_slot[ns] = next;
            c.stage_dec[ns] = dl;
            ++ns;
            ++next;
          }
        c.n_stage = ns;
        for (uint32_t k = 0; k < ns; ++k) c.slot_dec[c.stage_slot[k]] = c.stage_dec[k];
        for (uint32_t k = 0; k < slots; ++k) c.used[k] = 0;
      }
      __syncthreads();
      // every thread copies 16-byte pieces of the staged decoders
      const uint32_t ns = c.n_stage;
      for (uint32_t k = 0; k < ns; ++k) {
        const u32x4 *src = (const u32x4 *)(a.params + (size_t)c.stage_dec[k] * stride);
        u32x4 *dst = (u32x4 *)(wcache + (size_t)c.stage_slot[k] * stride);
        for (uint32_t i = tid; i < stride / 8; i += kFmaLdsThreads) dst[i] = src[i];
      }
      __syncthreads();
      if (pending && slot < 0)
        for (uint32_t k = 0; k < slots; ++k)
          if (c.slot_dec[k] == d) slot = (int)k;
      if (pending && slot >= 0) {
        pending = false;
        const uint16_t *p = wcache + (size_t)slot * stride;
        uint32_t h[32], o[32];
        fma_hidden_lds<S::F>(p, x, h, leaky, a.slope_h2);
        p += 64 * (S::F + 1);
        for (int l = 0; l < a.n_hidden; ++l) {
          fma_hidden_lds<64>(p, h, o, leaky, a.slope_h2);
#pragma unroll
          for (int i = 0; i < 32; ++i) h[i] = o[i];
          p += 64 * 65;
        }
        float y[16];
        fma_out_lds(p, a.out_dim, h, y);
        const int out_dim = a.out_dim;
        if (a.out_f16) {
          u32x2 *o2 = (u32x2 *)((uint16_t *)a.out + (size_t)q * out_dim);
#pragma unroll
          for (int cc = 0; cc < 16; cc += 4)
            if (cc < out_dim)
              o2[cc / 4] = u32x2{pack_half2(y[cc], y[cc + 1]), pack_half2(y[cc + 2], y[cc + 3])};
        } else {
          floatx4 *o4 = (floatx4 *)((float *)a.out + (size_t)q * out_dim);
#pragma unroll
          for (int cc = 0; cc < 16; cc += 4)
            if (cc < out_dim) o4[cc / 4] = floatx4{y[cc], y[cc + 1], y[cc + 2], y[cc + 3]};
        }
      }
    }
  }
}

// Compute units of the current device (one LDS-cache workgroup each).
inline int device_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus < 1)
    return 256;
  return cus;
}

template <int NL, int CH, int PE, bool MIP>
int launch_fma_lds(const DecodeArgs &a, uint32_t slots, hipStream_t stream) {
  const void *fn = (const void *)decode_fma_lds<NL, CH, PE, MIP>;
  const size_t lds = (size_t)slots * (size_t)a.dec_stride * sizeof(uint16_t);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return NTC_ERR_HIP;
  const uint64_t n_tiles = ((uint64_t)a.n + kFmaLdsThreads - 1) / kFmaLdsThreads;
  static const int cus = device_cus();
  const uint64_t groups = n_tiles < (uint64_t)cus ? n_tiles : (uint64_t)cus;
  hipLaunchKernelGGL((decode_fma_lds<NL, CH, PE, MIP>), dim3((unsigned)groups),
                     dim3(kFmaLdsThreads), lds, stream, a, slots, (uint32_t)n_tiles);
  return hip_status(hipGetLastError());
}

// Hidden width 64 takes the LDS weight cache when at least one decoder fits it;
// other shapes read their weights through the caches (decode_fma).
template <int NL, int CH, int PE, int HID, bool MIP>
int launch_fma_any(const DecodeArgs &a, hipStream_t stream) {
  if constexpr (HID == 64) {
    const size_t bytes = (size_t)a.dec_stride * sizeof(uint16_t);
    size_t slots = kFmaLdsWeightBytes / bytes;
    if (slots > kFmaMaxSlots) slots = kFmaMaxSlots;
    if (slots >= 1 && a.fma_cache) return launch_fma_lds<NL, CH, PE, MIP>(a, (uint32_t)slots, stream);
  }
  return launch_fma<NL, CH, PE, HID, MIP>(a, stream);
}

template <int NL, int CH, int PE, int HID>
int launch_fma_mip(const DecodeArgs &a, hipStream_t stream) {
  if constexpr (PE > 0) {
    return a.mip ? NTC_ERR_UNSUPPORTED : launch_fma_any<NL, CH, PE, HID, false>(a, stream);
  } else {
    return a.mip ? launch_fma_any<NL, CH, PE, HID, true>(a, stream)
                 : launch_fma_any<NL, CH, PE, HID, false>(a, stream);
  }
}

}  // namespace
}  // namespace ntc
