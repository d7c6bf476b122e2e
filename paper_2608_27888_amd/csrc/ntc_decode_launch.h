// ntc_decode_launch.h -- launches of the decode kernels of one decoder shape
// family: the kernel chosen by mode (binned, stream, per-wave stream), output
// store mode and activation.  Included by the per-family translation units.
#pragma once

#include "ntc_decode16.h"

namespace ntc {
namespace {

// Workgroups of `fn` that fill the current device at once (one round, no tail
// of late workgroups); *on_cu: those of one CU.
inline uint64_t resident_groups(const void *fn, int threads, size_t lds, int *on_cu = nullptr) {
  int dev = 0, cus = 256, per_cu = 0;
  if (hipGetDevice(&dev) == hipSuccess)
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  if (on_cu) *on_cu = per_cu;
  return (uint64_t)cus * (uint64_t)per_cu;
}

// Lets a kernel use more than the default 64 KB of dynamic LDS.
inline bool allow_lds(const void *fn, size_t lds) {
  return lds <= 64 * 1024 || hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)lds) == hipSuccess;
}

template <int NL, int CH, int PE, int HID, int NH, bool MIP, int STORE, bool LEAKY>
int launch_shape(const DecodeArgs &a, hipStream_t stream) {
  using N = Net<NL, CH, PE, HID, NH>;
  if (a.gather == NTC_GATHER_STAGED) {
    // the LDS-staged gather: binned, no mip blending, 2 levels, widths up to 8
    // (checked by the caller)
    if constexpr (!MIP && NL == 2 && !kWideRows<STORE>)
      if (a.bin_offset && a.out_dim <= 8) return launch_binned16<NL, CH, PE, HID, NH, STORE, LEAKY>(a, stream);
    return NTC_ERR_UNSUPPORTED;
  }
  const uint64_t tiles = a.bin_offset ? (uint64_t)a.max_tiles : ((uint64_t)a.n + kWave - 1) / kWave;
  if (tiles == 0) return NTC_OK;
  uint64_t blocks = (tiles + kWaves - 1) / kWaves;
  const uint32_t image_bytes = ((uint32_t)N::kImageBytes + 15u) & ~15u;
  if (a.bin_offset) {
    const void *fn = (const void *)decode_binned<NL, CH, PE, HID, NH, MIP, STORE, LEAKY>;
    if (!allow_lds(fn, image_bytes)) return NTC_ERR_HIP;
    int on_cu = 0;
    const uint64_t cap = resident_groups(fn, kThreads, image_bytes, &on_cu);
    if (blocks > cap) blocks = cap;
    // two workgroups on every CU (the grid a multiple of 16)
    const bool split = on_cu == 2 && blocks == cap && blocks % 16 == 0;
    hipLaunchKernelGGL((decode_binned<NL, CH, PE, HID, NH, MIP, STORE, LEAKY>),
                       dim3((unsigned)blocks), dim3(kThreads), image_bytes, stream, a,
                       split ? 1u : 0u);
  } else if constexpr (kRegWeights<HID>) {
    const void *fn = (const void *)decode_stream_reg<NL, CH, PE, HID, NH, MIP, STORE, LEAKY>;
    const uint64_t cap = resident_groups(fn, kThreads, 0);  // workgroups of kWaves
    // Waves share nothing but the decoder cache, so a call that does not fill the
    // chip takes narrower workgroups, without one, and reaches every CU (65,536
    // queries: 128 workgroups of 8 waves sit on half of the 256 CUs).
    uint64_t waves = kWaves;
    while (waves > 1 && tiles <= cap * waves / 2) waves /= 2;
    blocks = (tiles + waves - 1) / waves;
    if (blocks > cap * (kWaves / waves)) blocks = cap * (kWaves / waves);
    // the decoder cache takes a CU's LDS, so it goes with the widest workgroups
    // (one per CU anyway) and pays only where there is a decoder to switch to
    const bool cached = waves == kWaves && a.n_decoders > 1;
    const size_t lds = cached ? (size_t)RegNet<NL, CH, PE, HID, NH>::kSlots * N::kImageBytes : 0;
    if (!allow_lds(fn, lds)) return NTC_ERR_HIP;
    hipLaunchKernelGGL((decode_stream_reg<NL, CH, PE, HID, NH, MIP, STORE, LEAKY>),
                       dim3((unsigned)blocks), dim3((unsigned)waves * kWave), lds, stream, a,
                       cached ? 1u : 0u);
  } else {
    const void *fn = (const void *)decode_stream_mixed<NL, CH, PE, HID, NH, MIP, STORE, LEAKY>;
    const size_t lds = image_bytes + kWaves * N::kBiases * sizeof(float);
    if (!allow_lds(fn, lds)) return NTC_ERR_HIP;
    const uint64_t cap = resident_groups(fn, kThreads, lds);
    if (blocks > cap) blocks = cap;
    hipLaunchKernelGGL((decode_stream_mixed<NL, CH, PE, HID, NH, MIP, STORE, LEAKY>),
                       dim3((unsigned)blocks), dim3(kThreads), lds, stream, a, image_bytes);
  }
  return hip_status(hipGetLastError());
}

template <int NL, int CH, int PE, int HID, int NH, bool MIP, bool LEAKY>
int launch_store(const DecodeArgs &a, hipStream_t stream) {
  if (a.out_dim == 3)
    return a.out_f16 ? launch_shape<NL, CH, PE, HID, NH, MIP, kStoreF16x3, LEAKY>(a, stream)
                     : launch_shape<NL, CH, PE, HID, NH, MIP, kStoreF32x3, LEAKY>(a, stream);
  if (a.out_dim != 4 && a.out_dim != 8)
    return a.out_dim > 8 ? launch_shape<NL, CH, PE, HID, NH, MIP, kStoreEachWide, LEAKY>(a, stream)
                         : launch_shape<NL, CH, PE, HID, NH, MIP, kStoreEach, LEAKY>(a, stream);
  return a.out_f16 ? launch_shape<NL, CH, PE, HID, NH, MIP, kStoreF16x4, LEAKY>(a, stream)
                   : launch_shape<NL, CH, PE, HID, NH, MIP, kStoreF32x4, LEAKY>(a, stream);
}

template <int NL, int CH, int PE, int HID, int NH, bool MIP>
int launch_act(const DecodeArgs &a, hipStream_t stream) {
  return a.leaky ? launch_store<NL, CH, PE, HID, NH, MIP, true>(a, stream)
                 : launch_store<NL, CH, PE, HID, NH, MIP, false>(a, stream);
}

// Positional-encoding kernels exist for the Sec. 4 setup's decoder only: one
// hidden -> hidden layer, no mip blending.
template <int NL, int CH, int PE, int HID, int NH>
int launch_mip(const DecodeArgs &a, hipStream_t stream) {
  if constexpr (PE > 0) {
    return a.mip ? NTC_ERR_UNSUPPORTED : launch_act<NL, CH, PE, HID, NH, false>(a, stream);
  } else {
    return a.mip ? launch_act<NL, CH, PE, HID, NH, true>(a, stream)
                 : launch_act<NL, CH, PE, HID, NH, false>(a, stream);
  }
}

template <int NL, int CH, int PE, int HID>
int launch_hidden(const DecodeArgs &a, hipStream_t stream) {
  switch (a.n_hidden) {
    case 1: return launch_mip<NL, CH, PE, HID, 1>(a, stream);
    case 2:
      if constexpr (PE > 0) return NTC_ERR_UNSUPPORTED;
      else return launch_mip<NL, CH, PE, HID, 2>(a, stream);
    default: return NTC_ERR_UNSUPPORTED;
  }
}

}  // namespace

// One decoder shape family: every kernel variant (hidden layers, mip, store
// mode, activation) of the MFMA engine, and of the FMA engine.  Each family
// is instantiated in a translation unit of its own so that they compile in
// parallel.
template <int NL, int CH, int PE, int HID>
int launch_decode_shape(const DecodeArgs &a, hipStream_t stream) {
  return launch_hidden<NL, CH, PE, HID>(a, stream);
}

template <int NL, int CH, int PE, int HID>
int launch_decode_fma_shape(const DecodeArgs &a, hipStream_t stream) {
  return launch_fma_mip<NL, CH, PE, HID>(a, stream);
}

}  // namespace ntc
