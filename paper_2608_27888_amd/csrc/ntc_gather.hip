// ntc_gather.hip -- the feature vectors of a query stream alone: the gather
// step of the decode (bilinear samples of the texture's latent levels,
// concatenated finest first, levels blended by mip; Sec. 1 "latent pyramids or
// grids"), without the MLP.  The rows are the very values the decode's MLP
// consumes: the same device functions compute them, interpolation in packed
// fp16.
//
// One wave per 64 queries, grid stride.  Each lane loads its query, its 2x2 taps
// per level as 16-byte pieces of texel rows and interpolates; the rows then pass
// through LDS (wave private, fp16) so that a store instruction writes 1 KB of
// consecutive row pieces, 16 bytes a lane (fp32 rows: the fp16 values widened,
// exactly).  What bounds it: the written rows (64 bytes a query at 2 x 16 fp16
// channels) and the L1's tap traffic.  Storing each lane's own row, 16 bytes
// every 64 or more, touched 32 lines an instruction: 67.4 us for the 1080p frame's fp16
// rows; through LDS, non-temporal, 31.4 us (fp32 rows 111 -> 50).  On inputs read for the
// first time the taps' way from memory bounds it: 67 -> 53.6 us.
#include "ntc_decode_kernels.h"

namespace ntc {
namespace {

// Rows of up to this many bytes (half of the eight L2s) are left in the caches for
// whoever reads them next: as fast alone (9.2 us for 262,144 fp16 rows) and with a
// product of the rows with a 32 x 64 matrix behind it 52.7 us against 59.3.  More are
// stored past the caches (non-temporal).  Their reader pays for it, 475 us against 414
// for a 1080p frame's 133 MB and that product, but the gather alone takes 31.4 us
// against 51.8 where calls alternate between buffers (32.6 into one), 50 against 70
// for 265 MB.
constexpr uint64_t kCachedRows = (uint64_t)16 << 20;

// NT: non-temporal rows.
template <int NL, int CH, bool MIP, bool F16, bool NT>
__global__ void __launch_bounds__(kBlock) gather_rows(const DecodeArgs a) {
  constexpr int F = NL * CH;           // features per row, a multiple of 8
  constexpr int kStride = F / 2 + 4;   // words of an LDS row: odd in 16-byte pieces, so the
                                       // lanes' rows start on different banks
  static_assert(F % 16 == 0, "an even number of 16-byte pieces a row");
  __shared__ __attribute__((aligned(16))) uint32_t rows[kWavesPerBlock][kWave * kStride];
  const uint32_t lane = lane_id();
  uint32_t *mine = rows[threadIdx.x / kWave];
  const uint64_t n_tiles = ((uint64_t)a.n + kWave - 1) / kWave;
  const uint64_t stride = (uint64_t)gridDim.x * kWavesPerBlock;
  for (uint64_t t = (uint64_t)blockIdx.x * kWavesPerBlock +
                    __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
       t < n_tiles; t += stride) {
    const uint64_t q0 = t * kWave;
    const Query qq = validate(a, load_query<NL, MIP>(a, (uint32_t)(q0 + lane), q0 + lane < a.n));
    uint32_t x[F / 2];
    gather<NL, CH, 0, MIP>(a, qq, x);  // an invalid query samples texture 0
    const uint64_t valid = ballot(qq.valid);
    // a wave's LDS operations execute in order: the previous tile's reads come
    // before these writes, and the reads below after them
#pragma unroll
    for (int k = 0; k < F / 8; ++k)
      *(u32x4 *)(mine + lane * kStride + 4 * k) =
          u32x4{x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    constexpr int P = F16 ? F / 8 : F / 4;  // 16-byte pieces of a row in memory
    u32x4 *out = (u32x4 *)a.out + q0 * P;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const uint32_t p = (uint32_t)i * kWave + lane, row = p / P, piece = p % P;
      u32x4 v;
      if constexpr (F16) {
        v = *(const u32x4 *)(mine + row * kStride + 4 * piece);
      } else {
        const u32x2 h = *(const u32x2 *)(mine + row * kStride + 2 * piece);
        const half2v lo = as_h2(h[0]), hi = as_h2(h[1]);
        v = __builtin_bit_cast(u32x4, floatx4{(float)lo[0], (float)lo[1], (float)hi[0], (float)hi[1]});
      }
      if ((valid >> row) & 1) {
        if constexpr (NT) __builtin_nontemporal_store(v, out + p);
        else out[p] = v;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

template <int NL, int CH, bool MIP, bool F16>
int launch_rows(const DecodeArgs &a, hipStream_t stream) {
  uint64_t blocks = ((uint64_t)a.n + kBlock - 1) / kBlock;
  if (blocks > 65536) blocks = 65536;  // grid stride beyond
  const dim3 grid((unsigned)blocks), block(kBlock);
  if ((uint64_t)a.n * (NL * CH * (F16 ? 2 : 4)) <= kCachedRows)
    hipLaunchKernelGGL((gather_rows<NL, CH, MIP, F16, false>), grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((gather_rows<NL, CH, MIP, F16, true>), grid, block, 0, stream, a);
  return hip_status(hipGetLastError());
}

template <int NL, int CH>
int launch_shape(const DecodeArgs &a, bool f16, hipStream_t stream) {
  if (a.mip)
    return f16 ? launch_rows<NL, CH, true, true>(a, stream)
               : launch_rows<NL, CH, true, false>(a, stream);
  return f16 ? launch_rows<NL, CH, false, true>(a, stream)
             : launch_rows<NL, CH, false, false>(a, stream);
}

}  // namespace

int launch_gather(const DecodeArgs &a, int n_levels, int channels, bool f16, hipStream_t stream) {
  if (n_levels == 2 && channels == 8) return launch_shape<2, 8>(a, f16, stream);
  if (n_levels == 2 && channels == 16) return launch_shape<2, 16>(a, f16, stream);
  if (n_levels == 3 && channels == 16) return launch_shape<3, 16>(a, f16, stream);
  return NTC_ERR_UNSUPPORTED;
}

}  // namespace ntc
