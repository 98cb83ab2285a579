// wc_internal.h -- definitions shared by the host half (wc_host.cpp) and the
// device half (wc_decode.hip) of libwc.  Not part of the public ABI.
#pragma once

#include <stdint.h>

#include <mutex>
#include <vector>

#include "../../include/wc.h"

namespace wc {

constexpr uint32_t kMagic = 0x31424357u;  // "WCB1"
constexpr uint32_t kVersion = 5;        // blob format version
constexpr uint32_t kProbBits = 12;        // b = 12 (Sec. VI-F)
constexpr uint32_t kTableSize = 1u << kProbBits;
constexpr uint32_t kStateLow = 1u << 16;  // lower end of the state interval
constexpr uint32_t kHeaderBytes = 64;
constexpr uint32_t kDescBytes = 96;
constexpr uint32_t kMaxLanes = 64;
constexpr int kWideWaves = 16;  // waves to a workgroup of the 16-bit decode kernel

// The 16-wave decode kernel for bf16 / fp16 tensors in untiled 64-lane chunks
// (wc_decode_wide.hip): the waves of it resident on the current device at
// once (0 when unknown), and a launch of it with wc_decode's launch arguments
// (`bytes` their size; false on a launch error).
uint64_t wide_resident_waves();
bool wide_launch(const void* launch_args, uint64_t bytes, uint32_t workgroups, void* stream);
// The same for the fused decode-GEMM on 16-row tiles with up to 16 rows of x
// (wc_gemm_wide.hip); kind: 0 int8, 1 fp8 e4m3, 2 fp8 e5m2 weights, 3 MXFP4
// and 4 int4 codes coded as bytes, 5 bf16 weights (0 resident waves, or
// false, for any other kind).
uint64_t gemv_wide_resident_waves(int kind);
bool gemv_wide_launch(int kind, const void* launch_args, uint64_t bytes, uint32_t workgroups,
                      void* stream);
// kind 5 of the two above (wc_gemm_wide_bf16.hip)
uint64_t gemv_wide_bf16_resident_waves();
bool gemv_wide_bf16_launch(const void* launch_args, uint64_t bytes, uint32_t workgroups,
                           void* stream);

inline bool dtype_ok(uint32_t dt) { return dt >= WC_BF16 && dt <= WC_FP4_E2M1; }
inline bool has_raw(uint32_t dt) { return dt == WC_BF16 || dt == WC_FP16; }
// one symbol per byte (int8, fp8) / per nibble, low first (int4, fp4)
inline bool is_byte(uint32_t dt) { return dt == WC_U8 || dt == WC_FP8_E4M3 || dt == WC_FP8_E5M2; }
inline bool is_nibble(uint32_t dt) { return dt == WC_U4 || dt == WC_FP4_E2M1; }
inline uint32_t alphabet_of(uint32_t dt) { return is_nibble(dt) ? 16u : 256u; }
// W: symbols per lane-group; a lane-group is always 16 decoded bytes.
inline uint32_t group_of(uint32_t dt) { return is_nibble(dt) ? 32u : (is_byte(dt) ? 16u : 8u); }
inline uint64_t symbols_of(uint32_t dt, uint64_t bytes) {
  return is_nibble(dt) ? 2 * bytes : (is_byte(dt) ? bytes : bytes / 2);
}
inline uint64_t pad16(uint64_t x) { return (x + 15) & ~uint64_t(15); }

// Start states that carry data (blob version 4).  The encoder's start state
// comes back to the decoder for free at the end of a lane, so an untiled
// chunk spends it: lane l starts at 2^S + D, D packing the lane's first K
// symbols (b bits each, the first lowest), and those steps are not coded.  A
// decoded lane must end at 2^S + D with D within the symbols it carries.
// Tiled chunks, the fused GEMMs' input, start at 2^16 and carry nothing.
struct Carry {
  uint32_t K, b, S;
};
inline Carry carry_of(uint32_t dt, bool tiled) {
  if (tiled) return {0, 8, 16};
  if (has_raw(dt)) return {2, 8, 16};    // exponent bytes of bf16 / fp16
  if (is_nibble(dt)) return {7, 4, 28};  // int4 / fp4 nibbles
  return {3, 8, 24};                     // int8 / fp8 bytes
}
inline bool pow2(uint64_t x) { return x && !(x & (x - 1)); }

// A tensor is cut into tile_r x tile_c tiles (one chunk each) when its shape
// is divided exactly, tile_c is a power of two covering whole lane-groups,
// and a tile's decoded bytes are a valid chunk size; the column-block order
// also needs tile_r to be a power of two.
inline uint64_t tile_bytes(uint32_t dt, uint32_t tr, uint32_t tc) {
  return uint64_t(tr) * tc * 16 / group_of(dt);
}
inline bool tile_ok(uint32_t dt, uint64_t rows, uint64_t cols, uint32_t tr, uint32_t tc,
                    uint32_t order) {
  if (!tr || !tc || !rows || !cols || rows % tr || cols % tc || !pow2(tc) || tc < group_of(dt))
    return false;
  if (order > WC_TILE_COLUMN_BLOCKS || (order == WC_TILE_COLUMN_BLOCKS && !pow2(tr))) return false;
  const uint64_t cb = tile_bytes(dt, tr, tc);
  return cb >= 256 && cb <= (1u << 20) && cb % 256 == 0;
}

struct TensorInfo {
  uint32_t dtype = 0, chunk_bytes = 0, lanes = 0, group = 0, alphabet = 0;
  uint32_t tile_r = 0, tile_c = 0;  // 0, 0: chunks are byte runs
  uint32_t tile_order = 0;          // WC_TILE_ROWS or WC_TILE_COLUMN_BLOCKS
  uint64_t n_sym = 0, out_bytes = 0, first_chunk = 0, n_chunks = 0;
  uint64_t freq_off = 0, raw_off = 0, rows = 0, cols = 0;
  uint64_t sym_per_chunk() const { return symbols_of(dtype, chunk_bytes); }
};

struct BlobPriv {
  std::vector<uint8_t> bytes;
  std::vector<uint64_t> out_bytes;
  std::vector<TensorInfo> tensors;
  // raw regions at [raw_off, records_off), records at [records_off, size)
  uint64_t n_chunks = 0, index_off = 0, raw_off = 0, records_off = 0, size = 0;
};

// Which kernel decodes a launch (wc_decode.hip), from what its tensors add up to
// and the device's compute units and resident waves.
//
// The small kernel is for launches whose workgroups all run at once, one of eight
// chunks to a compute unit: what counts is its workgroups, not its chunks, because
// every tensor's last one may be short.  30 tensors of 65 chunks (1950 chunks in 270
// workgroups, 256 compute units) take 127 us on the general kernel and 161 in two
// rounds of small workgroups (64 KiB int8 chunks; bf16 74 and 77, int4 234 and 242).
// With up to four chunks to a compute unit its workgroups are of four: two fit a
// compute unit, so 32 short ones more are no second round.
//
// Chunks of fewer than kSmallSteps steps are over before the feeders have paid for
// their start: 1024 bf16 chunks of 8 steps take 8.4 us there and 7.9 on the general
// kernel, int8 chunks of 16 steps 8.9 and 8.5, of 32 steps 9.8 and 10.0.
//
// Two decodes at once, on two streams, bound the small kernel by its LDS accesses, of
// which a step has more than one of the general kernel (the feeders' lookups, one for
// every word): two launches of 1792 chunks together / one alone, general and small,
// 64 KiB int8 chunks 117 and 150 / 97 and 83 us, bf16 80 and 88 / 62 and 48, int4 215
// and 224 / 181 and 123; of 1340, 116 and 119 / 97 and 82, 75 and 71 / 61 and 47,
// 214 and 176 / 180 and 122; of 2040, bf16 79 and 94 / 61 and 49, int4 216 and 243 / 181
// and 124.  It ends about where two lose what a launch alone gains: int8, with the most
// words to a step, at 5.5 chunks to a compute unit, and so 16-bit chunks of fewer than
// kLongSteps steps (1700 of 16 KiB: 36 and 43 / 27 and 23 us), the others at 8.
//
// Column-block tiles of 64 rows and more are written 16 bytes a row at a time, which
// bounds any kernel (0.34 TB/s): up to four chunks to a compute unit the small one is
// still the faster (64 x 512 bf16, 1024 tiles 200 us against 203), above it is not
// (1280 tiles 252 and 246, 2048 tiles 395 and 382; 64 x 2048 int4, 1152 tiles 236 and
// 227).  Tiles of 32 rows keep it (32 x 1024 bf16, 2048 tiles 139 and 181).
constexpr uint32_t kSmallChunks = 8, kFewChunks = 4, kSmallSteps = 32, kLongSteps = 256;
constexpr uint32_t kTallRows = 64;
// 88 = 4 x 22 = 5.5 x 16 = 8 x 11
constexpr uint32_t kTall = 22, kHeavy = 16, kLight = 11, kSmallWork = 88;

enum class DecodeKernel { kGeneral, kWide, kSmall, kFew };

struct DecodeCapacity {
  uint64_t cus, general, wide;  // compute units; resident waves of two kernels
};

struct DecodeLaunch {
  uint64_t chunks = 0, small_wgs = 0, work = 0;
  uint64_t steps = 0;  // of the longest chunk
  bool lanes64 = true, wide_fits = true;

  void add(const TensorInfo& T) {
    chunks += T.n_chunks;
    small_wgs += (T.n_chunks + kSmallChunks - 1) / kSmallChunks;
    const uint64_t symbols = T.n_sym < T.sym_per_chunk() ? T.n_sym : T.sym_per_chunk();
    if (symbols > steps * T.lanes) steps = (symbols + T.lanes - 1) / T.lanes;
    const bool heavy = is_byte(T.dtype) || (has_raw(T.dtype) &&
                                            T.sym_per_chunk() < uint64_t(kLongSteps) * T.lanes);
    const bool tall = T.tile_order == WC_TILE_COLUMN_BLOCKS && T.tile_r >= kTallRows;
    work += T.n_chunks * (tall ? kTall : heavy ? kHeavy : kLight);
    lanes64 = lanes64 && T.lanes == 64;
    wide_fits = wide_fits && has_raw(T.dtype) && T.lanes == 64 && !T.tile_r;
  }
  DecodeKernel kernel(const DecodeCapacity& cap) const {
    if (!lanes64) return DecodeKernel::kGeneral;
    if (wide_fits && cap.general && cap.wide > cap.general && chunks > cap.general &&
        chunks <= cap.wide)
      return DecodeKernel::kWide;
    if (steps < kSmallSteps) return DecodeKernel::kGeneral;
    if (chunks <= cap.cus * kFewChunks) return DecodeKernel::kFew;
    if (small_wgs <= cap.cus && work <= cap.cus * kSmallWork) return DecodeKernel::kSmall;
    return DecodeKernel::kGeneral;
  }
};

// A value per device, worked out at its first use and kept without an allocation: an
// entry point that promises none, and that no C++ exception may leave, asks for it.
// Past kDevices devices it is worked out on every call.
template <class V>
class PerDevice {
 public:
  template <class Make>
  V get(int dev, Make make) {
    if (dev < 0 || dev >= kDevices) return make();
    std::lock_guard<std::mutex> lock(mu_);
    if (!known_[dev]) {
      value_[dev] = make();
      known_[dev] = true;
    }
    return value_[dev];
  }

 private:
  static constexpr int kDevices = 64;
  std::mutex mu_;
  bool known_[kDevices] = {};
  V value_[kDevices] = {};
};

// What a wc_blob's `priv` points at: the public struct and the parsed blob.
struct BlobHandle {
  wc_blob pub;
  BlobPriv priv;
};

// The data-independent part of a blob's layout, shared by the host encoder
// (wc_encode) and the device encoder (wc_encode_device): per-tensor chunking
// and tiling, the table each tensor uses and where it sits, the chunk index,
// the raw regions (right after the index) and where the records start.  Only
// the records' sizes, and with them the index and the blob's end, depend on
// the coded data.
struct Plan {
  std::vector<TensorInfo> tensors;  // freq_off absolute; raw_off relative to the raw regions' start
  std::vector<uint32_t> owner;      // tensor whose table a tensor uses (itself unless a layer codebook)
  uint64_t n_chunks = 0, index_off = 0, raw_start = 0, records_off = 0;
  uint64_t raw_region_bytes = 0;    // sum of pad16(n_sym) over the 16-bit tensors
  uint64_t worst_record_bytes = 0;  // all records if every symbol emitted a word
};

// Validate the encoder parameters and tensor sizes (WC_EINVAL on any bad
// field; the tensors' pointers are the caller's to check) and lay out the blob.
wc_status plan_blob(const wc_tensor* ts, uint32_t n, const wc_params* p, Plan& out);

// Symbols of chunk c of T, its lane-state count and its largest record.
inline uint64_t chunk_symbols(const TensorInfo& T, uint64_t c) {
  const uint64_t per = T.sym_per_chunk(), s0 = c * per;
  return s0 >= T.n_sym ? 0 : (T.n_sym - s0 < per ? T.n_sym - s0 : per);
}
inline uint32_t chunk_states(const TensorInfo& T, uint64_t n_c) {
  const uint64_t a = (n_c + T.group - 1) / T.group;
  return uint32_t(a < T.lanes ? a : T.lanes);
}
inline uint64_t worst_record(const TensorInfo& T, uint64_t n_c) {
  return 16 + pad16(4ull * chunk_states(T, n_c)) + pad16(2ull * n_c);
}

// Fill the rest of *out from out->hist (the field histograms of a tensor of
// dtype dt with n symbols) and, for 16-bit formats, the whole-word counts
// `joint16` (NULL otherwise; n_joint of them, in the order of their words, those
// that are zero left out or not): entropies, bounds, joint entropy.
void finish_stats(uint32_t dt, uint64_t n, const uint64_t* joint16, uint32_t n_joint,
                  wc_stats* out);
// Add the 65 536 whole-word counts of a 16-bit format, u64 from joint16 on or
// (narrow) u32 in the upper half of those 512 KiB, into out->hist[0] (coded field,
// bits 14..7) and out->hist[1] (raw field, bit 15 and bits 6..0), and move those
// that are not zero to the front as u64, in order; returns how many.
uint32_t split_word_counts(uint64_t* joint16, bool narrow, wc_stats* out);

// Validate `size` bytes at `p` and describe them.  Host-side checks of every
// header field, table sum and index entry; WC_EINVAL on the first failure.
wc_status parse_blob(const uint8_t* p, uint64_t size, BlobPriv& out);

}  // namespace wc
