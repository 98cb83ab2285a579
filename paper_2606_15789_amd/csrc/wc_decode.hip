// wc_decode.hip -- wc_decode: one launch decodes every chunk of a blob's
// tensors into the caller's buffers (Alg. 2; the decoder is in wc_decoder.h).
// The general kernel and the one for few chunks are here; bf16/fp16 launches
// that just overflow the general kernel's resident waves run on the 16-wave
// kernel of wc_decode_wide.hip.
#include "wc_decoder.h"

namespace {

using wc::kFewChunks;
using wc::kSmallChunks;

__global__ __launch_bounds__(kThreads) void wc_decode_kernel(LaunchArgs a) {
  __shared__ uint2 tab[wc::kTableSize];
  __shared__ uint32_t cum[260];
  __shared__ uint32_t ring[kWaves][wc_ring_words() / 2];
  const uint32_t wg = xcd_order(blockIdx.x, gridDim.x);
  // read where they are used: held together across twelve decoders, the fields
  // spilled 14 scalar registers
  const DevTensor& T = a.t[tensor_index(a, wg)];
  const WaveOf w = wave_of(a, T, wg, kWaves, T.lanes == 32 ? 2u : 1u);
  auto build = [&] {
    build_table(a, T, tab, cum, threadIdx.x);
    __syncthreads();
  };
  // instantiate one decoder per (format, lanes, tiling)
  auto run = [&](auto gc, auto lc) {
    constexpr int G = decltype(gc)::value, L = decltype(lc)::value;
    if (T.tiled)
      decode_chunks<G, L, true>(a, T, w.chunk, w.lane, tab, ring[w.wave], w.pre, build);
    else
      decode_chunks<G, L, false>(a, T, w.chunk, w.lane, tab, ring[w.wave], w.pre, build);
  };
  auto by_kind = [&](auto lc) {
    switch (T.kind) {
      case kSplit16: run(std::integral_constant<int, 2>{}, lc); break;
      case kByte: run(std::integral_constant<int, 4>{}, lc); break;
      default: run(std::integral_constant<int, 8>{}, lc); break;
    }
  };
  if (T.lanes == 32)
    by_kind(std::integral_constant<int, 32>{});
  else
    by_kind(std::integral_constant<int, 64>{});
}

// Launches of few 64-lane chunks: waves 0 .. kChunks - 1 decode a chunk each in
// steps of one LDS round trip, fed by the others (wc_ring.h).  Bound by the
// chain of a chunk's steps.  Rings of 1024 entries leave LDS for one workgroup of
// eight chunks, or two of four, to a compute unit: eight chunks, which is where
// the kernel ends (wc::DecodeLaunch), since with more the general kernel's 24 waves
// win (8B int8, 3332 chunks of 1024 steps: 135 us there, 168 to 185 us here).  On an
// 8 MB bf16 projection (128 chunks of 512 steps) a call takes 36 us against 54 on
// the general kernel, on the 8B int4 layer (1718 of 2048 steps) 125 against
// 187, on 16 ragged fp8 tensors (1355 of 512 steps) 46 against 56.  With up to four
// chunks to a compute unit, workgroups of four have a SIMD for each decoding wave
// (128 chunks of 64 KiB of another bf16 draw: 42 us, against 45 in workgroups of
// eight).
template <int kChunks>
__global__ __launch_bounds__(kChunks * 128) void wc_decode_small_kernel(LaunchArgs a) {
  // the table at LDS address 0 (a slot times 8 is its entry's address), then the
  // rings; the prefix sums the table is built from lie in the first ring, which
  // is filled after the build
  constexpr uint32_t kRings = 8u * wc::kTableSize;
  static_assert(260 * 4 <= kRingWritten, "the prefix sums fit the first ring");
  __shared__ __align__(16) uint8_t smem[kRings + kChunks * kRingWaveBytes];
  const uint32_t wg = xcd_order(blockIdx.x, gridDim.x);
  const DevTensor T = tensor_of(a, wg);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lane = __lane_id();
  const bool feeder = wave >= kChunks;
  const uint32_t slot = feeder ? wave - kChunks : wave;
  const uint32_t chunk = (wg - T.wg0) * kChunks + slot;
  const IndexPre pre = load_index(a, T, chunk, 1u);
  uint2* tab = reinterpret_cast<uint2*>(smem);
  uint32_t* ring = reinterpret_cast<uint32_t*>(smem + kRings + slot * kRingWaveBytes);
  auto build = [&] {
    build_table<kChunks * 128>(a, T, tab, reinterpret_cast<uint32_t*>(smem + kRings),
                                    threadIdx.x);
    __syncthreads();
  };
  if (feeder) {
    const uint32_t group = T.kind == kSplit16 ? 8u : (T.kind == kByte ? 16u : 32u);
    const Chain<64> c =
        open_chain<64, true>(a, T, min(chunk, T.n_chunks - 1u), group, lane, ring, pre);
    feed(c.rs, c.wbase[0], __builtin_amdgcn_readfirstlane(lds_address(ring)), lane, build);
    return;
  }
  auto run = [&](auto gc) {
    constexpr int G = decltype(gc)::value;
    if (T.tiled)
      decode_chunks<G, 64, true, 0, 0, 16, false, 0, FedRing>(a, T, chunk, lane, tab, ring, pre,
                                                           build);
    else
      decode_chunks<G, 64, false, 0, 0, 16, false, 0, FedRing>(a, T, chunk, lane, tab, ring, pre,
                                                            build);
  };
  switch (T.kind) {
    case kSplit16: run(std::integral_constant<int, 2>{}); break;
    case kByte: run(std::integral_constant<int, 4>{}); break;
    default: run(std::integral_constant<int, 8>{}); break;
  }
}

// The current device's compute units, and the waves of the general kernel and of the
// 16-bit wide kernel resident on it at once, from the runtime's occupancy calculation,
// worked out once per device (zeros when unknown: the general kernel is used).
wc::DecodeCapacity capacity() {
  static wc::PerDevice<wc::DecodeCapacity> known;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return {0, 0, 0};
  return known.get(dev, [&]() -> wc::DecodeCapacity {
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, reinterpret_cast<const void*>(wc_decode_kernel), kThreads, 0) != hipSuccess)
      return {0, 0, 0};
    return {uint64_t(cus), uint64_t(cus) * uint64_t(per_cu) * uint64_t(kWaves),
            wc::wide_resident_waves()};
  });
}

// A tiled tensor whose widest output descriptor (two tiles of a 32-lane wave)
// would not fit the 32-bit range the buffer descriptors address.
bool tile_span_ok(const wc::TensorInfo& T) {
  if (!T.tile_r) return true;
  const uint64_t pitch = T.cols * 16 / T.group;
  return (2 * uint64_t(T.tile_r) + 1) * pitch < (1ull << 31);
}

}  // namespace

extern "C" wc_status wc_decode(const wc_blob* desc, const void* dev_blob, void* const* dev_dst,
                               uint32_t n, void* stream, int32_t* dev_err) {
  if (!desc || !desc->priv || n != desc->n_tensors || (!dev_dst && n)) return WC_EINVAL;
  if (!dev_blob) return WC_EINVAL;
  const wc::BlobPriv& P = static_cast<const wc::BlobHandle*>(desc->priv)->priv;
  for (uint32_t t = 0; t < n; t++) {
    const wc::TensorInfo& T = P.tensors[t];
    if (T.n_chunks == 0) continue;
    if (T.lanes != 64 && T.lanes != 32) return WC_EUNSUPPORTED;
    if (!tile_span_ok(T)) return WC_EUNSUPPORTED;
    if (!dev_dst[t]) return WC_EINVAL;
  }
  LaunchArgs args{};
  fill_common(args, P, dev_blob, dev_err);
  uint32_t t = 0;
  while (t < n) {
    // the tensors of one launch: the next kMaxLaunchTensors that have chunks
    uint32_t end = t, nt = 0;
    wc::DecodeLaunch launch;
    for (; end < n && nt < kMaxLaunchTensors; end++) {
      const wc::TensorInfo& T = P.tensors[end];
      if (T.n_chunks == 0) continue;
      nt++;
      launch.add(T);
    }
    if (nt == 0) break;
    using wc::DecodeKernel;
    const DecodeKernel kernel =
        launch.lanes64 ? launch.kernel(capacity()) : DecodeKernel::kGeneral;
    const uint64_t waves = kernel == DecodeKernel::kWide    ? uint64_t(wc::kWideWaves)
                           : kernel == DecodeKernel::kFew   ? uint64_t(kFewChunks)
                           : kernel == DecodeKernel::kSmall ? uint64_t(kSmallChunks)
                                                            : uint64_t(kWaves);
    uint32_t wgs = 0;
    nt = 0;
    for (; t < end; t++) {
      const wc::TensorInfo& T = P.tensors[t];
      if (T.n_chunks == 0) continue;
      fill_tensor(args.t[nt++], T, dev_dst[t], wgs);
      const uint64_t per_group = waves * (T.lanes == 32 ? 2u : 1u);
      wgs += (uint32_t)((T.n_chunks + per_group - 1) / per_group);
    }
    set_tensors(args, nt);
    const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    switch (kernel) {
      case DecodeKernel::kWide:
        if (!wc::wide_launch(&args, sizeof args, wgs, stream)) return WC_EHIP;
        continue;
      case DecodeKernel::kFew:
        hipLaunchKernelGGL(wc_decode_small_kernel<kFewChunks>, dim3(wgs), dim3(kFewChunks * 128), 0,
                           st, args);
        break;
      case DecodeKernel::kSmall:
        hipLaunchKernelGGL(wc_decode_small_kernel<kSmallChunks>, dim3(wgs),
                           dim3(kSmallChunks * 128), 0, st, args);
        break;
      case DecodeKernel::kGeneral:
        hipLaunchKernelGGL(wc_decode_kernel, dim3(wgs), dim3(kThreads), 0, st, args);
        break;
    }
    if (hipGetLastError() != hipSuccess) return WC_EHIP;
  }
  return WC_OK;
}
