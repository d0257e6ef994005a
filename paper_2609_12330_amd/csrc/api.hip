// Host side of the C ABI declared in include/ef_attention.h: argument
// validation (synchronous, before anything is enqueued), kernel selection,
// grid and workspace arithmetic.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "ef_attention.h"
#include "ef_device.hpp"
#include "ef_kernels.hpp"

namespace {

constexpr int kTileKeys = 64;        // key tile of the kernels; partitions are multiples of it
constexpr int kDecodeMaxRows = 8;    // the VALU split producer handles G*Sq <= 8 ...
constexpr int kDecodeValuRows = 4;   // ... and the split-KV paths give it G*Sq <= 4 (the MFMA
                                     // producer streams faster with more rows)
constexpr int kMaxGridYZ = 65535;
static_assert(ef::kCounterRegionBytes == EF_COUNTER_REGION_BYTES,
              "the counter region of the header is the kernels' one");

struct Shape {
  int B, Hq, Hkv, Sq, Skv, D;
  long long rows() const { return (long long)B * Hq * Sq; }
};

bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

ef_status check_shape(const Shape& s) {
  if (s.B < 0 || s.Sq < 0 || s.Skv < 0 || s.Hq < 1 || s.Hkv < 1) return EF_ERR_INVALID_SHAPE;
  if (s.Hq % s.Hkv != 0) return EF_ERR_GQA_RATIO;
  if (s.D != 64 && s.D != 128) return EF_ERR_UNSUPPORTED_HEAD_DIM;
  // Per-head extents stay below 2^31 elements; batch*heads fits the grid.
  if ((long long)s.Sq * s.D >= (1LL << 31) || (long long)s.Skv * s.D >= (1LL << 31))
    return EF_ERR_INVALID_SHAPE;
  if ((long long)s.B * s.Hkv > kMaxGridYZ || (long long)(s.Hq / s.Hkv) * s.Sq >= (1LL << 31))
    return EF_ERR_INVALID_SHAPE;
  return EF_OK;
}

ef_status check_io(const Shape& s, const void* q, const void* k, const void* v, const float* o,
                   float scale) {
  if (!std::isfinite(scale)) return EF_ERR_INVALID_SCALE;
  if (s.rows() == 0) return EF_OK;
  if (q == nullptr || o == nullptr) return EF_ERR_NULL_POINTER;
  if (s.Skv > 0 && (k == nullptr || v == nullptr)) return EF_ERR_NULL_POINTER;
  if (misaligned(q) || misaligned(o) || misaligned(k) || misaligned(v)) return EF_ERR_MISALIGNED;
  return EF_OK;
}

// Visible key runs of a (batch, kv head) for a causal window of `window` keys
// and `sinks` sink keys (section 7.3). Every key of every query row lies in
// the sink run [0, la) or the window run [bs, Skv): bs is the first key of the
// earliest row's window (row 0, diagonal Skv - Sq) rounded down to a tile, la
// the sink count rounded up to one. The split producers partition the
// concatenation of the two runs (lv keys). A window of at least Skv keys hides
// nothing beyond the causal mask and is dropped.
ef::KeyRuns key_runs(int Sq, int Skv, int window, int sinks) {
  ef::KeyRuns r{0, 0, Skv, 0, 0};
  if (window <= 0 || window >= Skv) return r;
  const int sk = sinks < Skv ? sinks : Skv;
  int la = (sk + kTileKeys - 1) / kTileKeys * kTileKeys;
  if (la > Skv) la = Skv;
  long long ws = (long long)Skv - Sq - window + 1;  // window start of row 0
  if (ws < 0) ws = 0;
  int bs = (int)(ws / kTileKeys * kTileKeys);
  if (bs < la) bs = la;
  r.la = la;
  r.bs = bs;
  r.lv = la + (Skv - bs);
  r.window = window;
  r.sinks = sk;
  return r;
}

// Roofline model of one split-KV call with T keys per partition (section 6.2,
// over the legal schedules, minimise the largest work/throughput ratio over
// the modelled resources). Resources: HBM (K/V, q, o and the partial states
// written and read back) and the streaming time of one workgroup (T keys of K
// and V, or the fewer keys its rows can see, at that workgroup's rate, times
// the rounds of workgroups the chip holds); the combine follows (inside the
// producer for up to 64 partitions, else a second kernel). The rates were fitted to partition-size sweeps of
// twelve decode shapes on MI355X (1 to 64 query rows per kv head, 1K to 128K
// keys): the VALU producer streams 6.5 TB/s over the chip and 27.6, 51.1 or
// 10.3 GB/s per workgroup for 1, 2 or 4 query rows per kv head (one, two and
// one waves), plus 5 us per round; the combine inside it costs 4.4 us per 16
// partitions, the combine kernel 8.9 us plus its reads. The MFMA producer
// streams 5.85 TB/s over the chip and 9.9 GB/s per wave, plus 1 us per round,
// and its combine kernel costs 13.4 us plus its reads. 2048 waves are resident.
// The chip's rate is reached only with enough waves streaming at once: under
// load a wave draws about 16 GB/s (VALU) or 8.5 GB/s (MFMA), counted over the
// waves weighted by their share of the keys (a short last partition adds
// little).
// The rates of 3 or 4 rows are those of one wave per partition, while up to 512
// partitions now run four (launch_decode_split) and take 9-70% less than modelled:
// over 142 decode shapes (1 to 16 sequences, 2 to 8 kv heads, 512 to 65536 keys) the
// pick is 5.4% slower than the best size in the mean, 28% at most (2 x 32/8 heads,
// 8192 keys: 64 keys 20.8 us, 512 keys 17.4). A model of both forms came within 1.6%
// on those shapes, but on 70 others the sizes it chose instead (mostly 2 to 8 times
// larger) were 1.3% faster in the mean and up to 25% slower, and fewer references
// mean more rounding: the error against 64 bits grew by 15% in the mean, 3.6 times
// where 64 keys had held 16 per wave. So the choice stays with the one-wave rates.
constexpr double kHbmValuBytesPerUs = 6.5e6;
constexpr double kHbmMfmaBytesPerUs = 5.85e6;
constexpr double kWgValuBytesPerUs[3] = {27.6e3, 51.1e3, 10.3e3};  // 1, 2, 4 rows
constexpr double kWaveMfmaBytesPerUs = 9.9e3;
constexpr double kLoadedWaveValuBytesPerUs = 16.0e3;
constexpr double kLoadedWaveMfmaBytesPerUs = 8.5e3;
constexpr double kResidentWaves = 2048.0;
constexpr double kRoundValuUs = 5.0;
constexpr double kRoundMfmaUs = 1.0;
constexpr double kFusedCombineUsPer16 = 4.4;
constexpr double kCombineValuUs = 8.9;
constexpr double kCombineMfmaUs = 13.4;

// Rows per workgroup of the matrix-core kernel (section 6.2). The legal
// schedules hold 64 or 128 query rows of one kv head (two or four waves of 32
// rows). Each is charged an optimistic time, the larger of its matrix work over
// the bf16 peak and its global-memory traffic over the HBM peak, and the
// fastest is taken; with equal times, the one with less matrix work. Matrix
// work counts the rows padded to whole workgroups; traffic counts the K/V that
// every row tile stages (each re-read in full: the L2 is not credited) plus q
// and o once. `keys`: the keys a row tile streams.
constexpr double kMfmaPeakFlopsPerUs = 2.5e9;
constexpr double kHbmPeakBytesPerUs = 8.0e6;

int rows_per_block(const Shape& s, double keys) {
  const double R = (double)(s.Hq / s.Hkv) * s.Sq;
  const double kv_heads = (double)s.B * s.Hkv;
  int best = 0;
  double best_us = 0.0, best_flops = 0.0;
  for (const int bm : {64, 128}) {
    const double tiles = std::ceil(R / bm);
    const double flops = kv_heads * tiles * bm * keys * 4.0 * s.D;
    const double bytes = kv_heads * tiles * keys * 4.0 * s.D + (double)s.rows() * s.D * 6.0;
    const double us = std::max(flops / kMfmaPeakFlopsPerUs, bytes / kHbmPeakBytesPerUs);
    if (best == 0 || us < best_us || (us == best_us && flops < best_flops)) {
      best = bm;
      best_us = us;
      best_flops = flops;
    }
  }
  return best;
}

double split_model_us(const Shape& s, int keys, int T, int visible) {
  const int G = s.Hq / s.Hkv;
  const int R = G * s.Sq;
  const double P = std::ceil((double)keys / T);
  const double Tk = std::min<double>(T, keys);
  // A workgroup streams at most the keys its rows can see, however long its partition.
  const double Twg = std::min<double>(Tk, visible);
  const bool valu = R <= kDecodeValuRows;
  double nw, wg_per_part, wg_rate;
  if (valu) {
    const int bucket = R <= 1 ? 0 : R <= 2 ? 1 : 2;
    nw = bucket == 1 ? 2 : 1;  // waves per workgroup of the VALU producer
    wg_per_part = 1;
    wg_rate = kWgValuBytesPerUs[bucket];
  } else {
    const int bm = rows_per_block(s, std::min<double>(T, visible));
    nw = bm / 32;
    wg_per_part = std::ceil((double)R / bm);
    wg_rate = kWaveMfmaBytesPerUs * nw;
  }
  const double kv_heads = (double)s.B * s.Hkv;
  const double rows = (double)s.B * s.Hq * s.Sq;
  const double kv_bytes = kv_heads * keys * s.D * 4.0;
  const double io_bytes = rows * s.D * 6.0;
  const double state_bytes = rows * P * (s.D + 2) * 4.0;
  const double hbm = valu ? kHbmValuBytesPerUs : kHbmMfmaBytesPerUs;
  const double waves = kv_heads * P * wg_per_part * nw;
  const double waves_eff = kv_heads * wg_per_part * nw * keys / Tk;
  const double hbm_eff =
      std::min(hbm, std::min(waves_eff, kResidentWaves) *
                        (valu ? kLoadedWaveValuBytesPerUs : kLoadedWaveMfmaBytesPerUs));
  const double r_hbm = (kv_bytes + io_bytes + 2.0 * state_bytes) / hbm_eff;
  const double rounds = std::ceil(waves / kResidentWaves);
  const double r_wg =
      rounds * (Twg * s.D * 4.0 / wg_rate + (valu ? kRoundValuUs : kRoundMfmaUs));
  const bool fused = valu && P <= ef::kFusedMaxP && kv_heads <= ef::kCounterSlots;
  const double combine = fused ? kFusedCombineUsPer16 * std::ceil(P / 16.0)
                               : state_bytes / hbm + (valu ? kCombineValuUs : kCombineMfmaUs);
  return std::max(r_hbm, r_wg) + combine;
}

// Candidate partition sizes for a key axis of `keys` keys: 64, 128, 256, 512,
// ... (powers of two times 64), up to one partition holding every key; at most
// 65535 partitions.
std::vector<int> partition_candidates(int keys) {
  std::vector<int> out;
  const long long top = ((long long)std::max(keys, 1) + kTileKeys - 1) / kTileKeys * kTileKeys;
  // Powers of two times the tile: sizes in between leave a ragged last
  // partition on power-of-two contexts and measured slower than both neighbours.
  for (long long t = kTileKeys; t < top; t *= 2)
    if ((keys + t - 1) / t <= kMaxGridYZ) out.push_back((int)t);
  out.push_back((int)top);
  std::sort(out.begin(), out.end());
  out.erase(std::unique(out.begin(), out.end()), out.end());
  return out;
}

// The most keys of the virtual key axis the rows of one workgroup can see: the
// whole axis without a window; with one, the sink run plus the union of the
// rows' windows. A workgroup of the matrix-core producer holds the rows of
// ceil(BM / G) query positions (rows are packed r = sq*G + g), one of the vector
// producer all Sq of them. A window run cut into partitions leaves each row
// tile most of its keys in one partition, so splitting it shortens no
// workgroup's stream (attention-sink prefill: 1024 positions, a 5,123-key run,
// 4,228 keys per row tile).
int visible_keys(const Shape& s, const ef::KeyRuns& runs) {
  if (runs.window <= 0) return runs.lv;
  const int G = s.Hq / s.Hkv;
  const int R = G * s.Sq;
  const int pos = R <= kDecodeValuRows
                      ? s.Sq
                      : std::min(s.Sq, (rows_per_block(s, runs.lv) + G - 1) / G);
  const long long v = (long long)runs.window + runs.sinks + pos;
  return (int)std::min<long long>(runs.lv, v);
}

// Keys per partition of a key axis of `keys` keys (the visible runs' length):
// the caller's choice, else the candidate the model rates fastest.
int resolve_partition(const Shape& s, int keys, int partition_size, int visible) {
  if (partition_size > 0) return partition_size;
  if (keys <= 0) return kTileKeys;
  int best = kTileKeys;
  double best_us = 1e300;
  for (int t : partition_candidates(keys)) {
    const double us = split_model_us(s, keys, t, visible);
    if (us < best_us) {
      best_us = us;
      best = t;
    }
  }
  return best;
}

ef_status check_mask(int window, int sinks) {
  return (window < 1 || sinks < 0) ? EF_ERR_INVALID_MASK : EF_OK;
}

struct WsLayout {
  size_t m_off, l_off, acc_off, cnt_off, bytes;
};

// Counters first (a region of fixed size, see kCounterRegionBytes), then the
// partial states.
WsLayout ws_layout(long long rows, long long P, int D) {
  WsLayout w;
  const size_t a = ef::ws_align256((size_t)(rows * P) * sizeof(float));
  w.cnt_off = 0;
  w.m_off = ef::kCounterRegionBytes;
  w.l_off = w.m_off + a;
  w.acc_off = w.m_off + 2 * a;
  w.bytes = w.acc_off + ef::ws_align256((size_t)(rows * P) * (size_t)D * sizeof(float));
  return w;
}

// Whether the producer combines the states itself: few query rows per kv head
// (the vector producer), few partitions, and a counter slot for every group.
bool fused_combine(const Shape& s, long long P, int d_splits) {
  return ((long long)(s.Hq / s.Hkv) * s.Sq <= kDecodeValuRows || d_splits > 0) &&
         P <= ef::kFusedMaxP &&
         (long long)s.B * s.Hkv * std::max(d_splits, 1) <= ef::kCounterSlots;
}

ef_status from_hip(hipError_t e) { return e == hipSuccess ? EF_OK : EF_ERR_HIP; }

// Whether a single-pass launch runs 64-row tiles whose key tiles two groups of
// waves share (MfmaParams::key_split). A launch with fewer workgroups than the
// chip holds waits for its longest chain of key tiles, which two groups halve;
// with more, the rows of a 128-row workgroup make better use of each staged
// tile. The two-group workgroup takes 128 KiB of LDS at D = 128 (one per CU) and
// 64 KiB at D = 64 (two), so the line is one round of them; causal launches whose
// workgroups get much shorter towards the end go a quarter past it (with a
// window, or few queries over a long context, they do not: 8/2 heads of 64, 5 x
// 865 of 4771 keys with a 792-key window [550] 25.6 / 26.4). Measured, one group
// of 64 or 128 rows against two groups (us; 64-row tiles in brackets): D = 128
// full, 4096^2 x 4 heads [256] 66.9 / 47.6; causal 1024 of 8192 keys x 16 heads
// [256] 127.0 / 87.0, 32/8 heads 640 [320] 17.7 / 16.8, 777 [392] 20.4 / 20.8,
// 16/4 heads 2048 [512] 39.5 / 41.8; 64 rows of 4000 keys x 32 [32] 63.2 / 45.7;
// D = 64, 4 x 16 heads 384 full [384] 10.2 / 9.8, 16 heads 2048 causal [512] 29.7
// / 23.6, 8 x 12 heads 384 full [576] 13.5 / 15.9.
bool use_key_split(const Shape& s, const ef::KeyRuns& runs, int causal) {
  const long long R = (long long)(s.Hq / s.Hkv) * s.Sq;
  const long long tiles = (long long)s.B * s.Hkv * ((R + 63) / 64);
  const long long slots = s.D == 128 ? 256 : 512;
  const bool short_tail = causal && runs.window == 0 && s.Skv <= 2LL * s.Sq;
  return runs.lv > kTileKeys && tiles <= (short_tail ? slots + slots / 4 : slots);
}

// Whether a single-pass launch visits its row tiles longest first over all heads
// of an XCD. Head by head, the last head's longest tiles start late and end the
// launch alone; this pays where causal tiles differ in length (few queries over
// a long context, or a window, make them nearly equal: 32 heads, 4096 of 16384
// keys, 4096-key window 272 -> 282 us) and as long as the K/V of an XCD's heads,
// which are then all in use at once, stay in the caches (4 MiB of L2 per XCD, 256
// MiB behind all of them). Head by head / longest first (us; MiB of K/V per XCD
// in brackets): causal, D = 128, 32/8 heads, 4 x 2048 145.9 / 144.3 [4], 4 x 4096
// 525.8 / 522.1 [8], 32 heads 2048 56.0 / 48.1 [4], 8192 517 / 497 [16], 4 x 2048
// 179 / 167 [16]; D = 64, 32 heads, 4 x 1024 38.8 / 31.7 [4], 16384 1118 / 1081
// [16]. Past that the order loses: D = 64, 16 x 12 heads 4096 483 / 492 [24]; D =
// 128, 4 x 32 heads 4096 570 / 590 [32], 4096 of 8192 1483 / 1817 [64], of 16384
// 3348 / 4430 [128], 16 x 12 heads 4096 850 / 989 [48].
constexpr long long kLongestFirstKvBytes = 16LL << 20;

bool longest_first(const Shape& s, const ef::KeyRuns& runs, int causal) {
  const long long kv_heads = (long long)s.B * s.Hkv;
  return causal && runs.window == 0 && s.Skv <= 4LL * s.Sq && kv_heads % ef::kXcds == 0 &&
         kv_heads / ef::kXcds * s.Skv * s.D * 4 <= kLongestFirstKvBytes;
}

// How a single-pass launch runs: query rows per workgroup, key tiles shared by two
// groups of waves, row tiles longest first.
struct FwdSchedule {
  int bm, key_split, interleave;
};

FwdSchedule fwd_schedule(const Shape& s, const ef::KeyRuns& runs, int causal) {
  const int split = use_key_split(s, runs, causal) ? 1 : 0;
  return {split ? 64 : rows_per_block(s, runs.lv), split, longest_first(s, runs, causal) ? 1 : 0};
}

ef_status launch_mfma(const Shape& s, const void* q, const void* k, const void* v, float* o,
                      float* ws_m, float* ws_l, float* ws_acc, int T, int P, float scale,
                      int causal, const ef::KeyRuns& runs, hipStream_t stream,
                      const void* q2 = nullptr, const void* k2 = nullptr,
                      const ef::DiffParams* diff = nullptr, int renew = 0) {
  ef::MfmaParams a{};
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const uint16_t*>(k);
  a.v = static_cast<const uint16_t*>(v);
  a.o = o;
  a.ws_m = ws_m;
  a.ws_l = ws_l;
  a.ws_acc = ws_acc;
  a.B = s.B; a.Hq = s.Hq; a.Hkv = s.Hkv; a.Sq = s.Sq; a.Skv = s.Skv; a.D = s.D;
  a.G = s.Hq / s.Hkv;
  a.R = a.G * s.Sq;
  a.T = T;
  a.P = P;
  a.bm = rows_per_block(s, std::min(T, runs.lv));
  a.c_abs = std::fabs(scale) * ef::kLog2e;
  a.qflip = scale < 0.f ? 0x80008000u : 0u;
  a.causal = causal ? 1 : 0;
  a.runs = runs;
  if (diff != nullptr) {
    a.q2 = static_cast<const uint16_t*>(q2);
    a.k2 = static_cast<const uint16_t*>(k2);
    a.diff = *diff;
    a.renew = renew;
  } else if (ws_m == nullptr) {
    const FwdSchedule f = fwd_schedule(s, runs, causal);
    a.bm = f.bm;
    a.key_split = f.key_split;
    a.interleave = f.interleave;
  }
  a.mtiles = (a.R + a.bm - 1) / a.bm;
  return from_hip(ef::launch_mfma_attention(a, stream));
}

}  // namespace

extern "C" {

int ef_abi_version(void) { return EF_ABI_VERSION; }

const char* ef_status_string(int status) {
  switch (status) {
    case EF_OK: return "ok";
    case EF_ERR_NULL_POINTER: return "a required pointer is NULL";
    case EF_ERR_INVALID_SHAPE: return "invalid shape (negative size, Hq or Hkv < 1, or too large)";
    case EF_ERR_GQA_RATIO: return "Hq is not a multiple of Hkv";
    case EF_ERR_UNSUPPORTED_HEAD_DIM: return "head dimension must be 64 or 128";
    case EF_ERR_MISALIGNED: return "a pointer is not 16-byte aligned";
    case EF_ERR_INVALID_PARTITION:
      return "partition_size must be 0 or a positive multiple of 64 giving at most 65535 "
             "partitions";
    case EF_ERR_WORKSPACE_TOO_SMALL: return "workspace is NULL or too small";
    case EF_ERR_INVALID_SCALE: return "scale is not finite";
    case EF_ERR_HIP: return "HIP error while enqueueing work";
    case EF_ERR_INVALID_MASK: return "window must be >= 1 and sinks >= 0";
    case EF_ERR_INVALID_DIFF: return "lambda_init and eps must be finite and eps >= 0";
    case EF_ERR_INVALID_SPLIT:
      return "d_splits must be 1, 2 or 4, with at most 8 query rows per kv head";
    case EF_ERR_SCRATCH_TOO_SMALL:
      return "the problem needs more workspace than the library's static scratch holds";
    default: return "unknown status";
  }
}

}  // extern "C"

namespace {

ef_status fwd_impl(const Shape& s, const void* q, const void* k, const void* v, float* o,
                   float scale, int causal, const ef::KeyRuns& runs, void* stream) {
  ef_status st = check_shape(s);
  if (st != EF_OK) return st;
  st = check_io(s, q, k, v, o, scale);
  if (st != EF_OK) return st;
  if (s.rows() == 0) return EF_OK;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (s.Skv == 0) return from_hip(ef::launch_zero_fill(o, (size_t)s.rows() * s.D, hs));
  return launch_mfma(s, q, k, v, o, nullptr, nullptr, nullptr, runs.lv, 1, scale, causal, runs,
                     hs);
}

// The split-KV entry points reject more partitions than the grid takes; the
// size queries report such arguments as invalid (0) too.
int partition_size_impl(const Shape& s, const ef::KeyRuns& runs, int partition_size) {
  if (check_shape(s) != EF_OK) return 0;
  if (partition_size < 0 || partition_size % kTileKeys != 0) return 0;
  const int T = resolve_partition(s, runs.lv, partition_size, visible_keys(s, runs));
  if ((runs.lv + (long long)T - 1) / T > kMaxGridYZ) return 0;
  return T;
}

size_t workspace_size_impl(const Shape& s, const ef::KeyRuns& runs, int partition_size) {
  if (check_shape(s) != EF_OK) return 0;
  if (partition_size < 0 || partition_size % kTileKeys != 0) return 0;
  if (s.rows() == 0 || s.Skv == 0) return 0;
  const int T = resolve_partition(s, runs.lv, partition_size, visible_keys(s, runs));
  const long long P = (runs.lv + (long long)T - 1) / T;
  if (P > kMaxGridYZ) return 0;
  return ws_layout(s.rows(), P, s.D).bytes;
}

}  // namespace

extern "C" {

ef_status ef_attention_fwd(const void* q, const void* k, const void* v, float* o, int B, int Hq,
                           int Hkv, int Sq, int Skv, int D, float scale, int causal,
                           void* stream) {
  return fwd_impl(Shape{B, Hq, Hkv, Sq, Skv, D}, q, k, v, o, scale, causal,
                  key_runs(Sq, Skv, 0, 0), stream);
}

ef_status ef_attention_fwd_local(const void* q, const void* k, const void* v, float* o, int B,
                                 int Hq, int Hkv, int Sq, int Skv, int D, float scale, int window,
                                 int sinks, void* stream) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  ef_status st = check_shape(s);
  if (st != EF_OK) return st;
  st = check_mask(window, sinks);
  if (st != EF_OK) return st;
  return fwd_impl(s, q, k, v, o, scale, 1, key_runs(Sq, Skv, window, sinks), stream);
}

int ef_attention_splitkv_partition_size(int B, int Hq, int Hkv, int Sq, int Skv, int D,
                                        int partition_size) {
  return partition_size_impl(Shape{B, Hq, Hkv, Sq, Skv, D}, key_runs(Sq, Skv, 0, 0),
                             partition_size);
}

size_t ef_attention_splitkv_workspace_size(int B, int Hq, int Hkv, int Sq, int Skv, int D,
                                           int partition_size) {
  return workspace_size_impl(Shape{B, Hq, Hkv, Sq, Skv, D}, key_runs(Sq, Skv, 0, 0),
                             partition_size);
}

int ef_attention_splitkv_local_partition_size(int B, int Hq, int Hkv, int Sq, int Skv, int D,
                                              int window, int sinks, int partition_size) {
  if (check_mask(window, sinks) != EF_OK) return 0;
  return partition_size_impl(Shape{B, Hq, Hkv, Sq, Skv, D}, key_runs(Sq, Skv, window, sinks),
                             partition_size);
}

size_t ef_attention_splitkv_local_workspace_size(int B, int Hq, int Hkv, int Sq, int Skv, int D,
                                                 int window, int sinks, int partition_size) {
  if (check_mask(window, sinks) != EF_OK) return 0;
  return workspace_size_impl(Shape{B, Hq, Hkv, Sq, Skv, D}, key_runs(Sq, Skv, window, sinks),
                             partition_size);
}

}  // extern "C"

namespace {

// Validation shared by the split-KV entry points; on success fills the
// partition count and the workspace pointers.
ef_status split_prepare(const Shape& s, const void* q, const void* k, const void* v,
                        const float* o, float scale, const ef::KeyRuns& runs,
                        int partition_size, void* workspace, size_t workspace_bytes, int* T_out,
                        int* P_out, float** ws_m, float** ws_l, float** ws_acc,
                        unsigned** counters) {
  ef_status st = check_shape(s);
  if (st != EF_OK) return st;
  if (partition_size < 0 || partition_size % kTileKeys != 0) return EF_ERR_INVALID_PARTITION;
  st = check_io(s, q, k, v, o, scale);
  if (st != EF_OK) return st;
  *T_out = 0;
  *P_out = 0;
  if (s.rows() == 0 || s.Skv == 0) return EF_OK;
  const int T = resolve_partition(s, runs.lv, partition_size, visible_keys(s, runs));
  const long long P = (runs.lv + (long long)T - 1) / T;
  if (P > kMaxGridYZ) return EF_ERR_INVALID_PARTITION;
  const WsLayout w = ws_layout(s.rows(), P, s.D);
  if (workspace == nullptr || workspace_bytes < w.bytes) return EF_ERR_WORKSPACE_TOO_SMALL;
  if (misaligned(workspace)) return EF_ERR_MISALIGNED;
  char* ws = static_cast<char*>(workspace);
  *ws_m = reinterpret_cast<float*>(ws + w.m_off);
  *ws_l = reinterpret_cast<float*>(ws + w.l_off);
  *ws_acc = reinterpret_cast<float*>(ws + w.acc_off);
  *counters = reinterpret_cast<unsigned*>(ws + w.cnt_off);
  *T_out = T;
  *P_out = (int)P;
  return EF_OK;
}

// Stores the partition states; with `counters` and `o` given (decode path only),
// the last workgroup of each (batch, kv head) also combines them into o.
// d_splits = 0 lets the row count choose the producer; d_splits >= 1 asks for
// the VALU producer with that many output-channel slices.
ef_status split_produce(const Shape& s, const void* q, const void* k, const void* v, float scale,
                        int causal, const ef::KeyRuns& runs, int T, int P, float* ws_m,
                        float* ws_l, float* ws_acc, unsigned* counters, float* o,
                        hipStream_t hs, int d_splits = 0) {
  const int G = s.Hq / s.Hkv;
  const int R = G * s.Sq;
  if (d_splits > 0 || R <= kDecodeValuRows) {
    ef::DecodeParams a{};
    a.q = static_cast<const uint16_t*>(q);
    a.k = static_cast<const uint16_t*>(k);
    a.v = static_cast<const uint16_t*>(v);
    a.ws_m = ws_m;
    a.ws_l = ws_l;
    a.ws_acc = ws_acc;
    a.B = s.B; a.Hq = s.Hq; a.Hkv = s.Hkv; a.Sq = s.Sq; a.Skv = s.Skv; a.D = s.D;
    a.G = G;
    a.R = R;
    a.T = T;
    a.P = P;
    a.c = scale * ef::kLog2e;
    a.causal = causal ? 1 : 0;
    a.counters = counters;
    a.o = o;
    a.runs = runs;
    a.d_splits = d_splits > 0 ? d_splits : 1;
    return from_hip(ef::launch_decode_split(a, hs));
  }
  return launch_mfma(s, q, k, v, nullptr, ws_m, ws_l, ws_acc, T, P, scale, causal, runs, hs);
}

ef_status splitkv_impl(const Shape& s, const void* q, const void* k, const void* v, float* o,
                       float scale, int causal, const ef::KeyRuns& runs, int partition_size,
                       void* workspace, size_t workspace_bytes, void* stream) {
  int T = 0, P = 0;
  float *ws_m = nullptr, *ws_l = nullptr, *ws_acc = nullptr;
  unsigned* counters = nullptr;
  ef_status st = split_prepare(s, q, k, v, o, scale, runs, partition_size, workspace,
                               workspace_bytes, &T, &P, &ws_m, &ws_l, &ws_acc, &counters);
  if (st != EF_OK || s.rows() == 0) return st;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (s.Skv == 0) return from_hip(ef::launch_zero_fill(o, (size_t)s.rows() * s.D, hs));
  if (fused_combine(s, P, 0))
    return split_produce(s, q, k, v, scale, causal, runs, T, P, ws_m, ws_l, ws_acc, counters, o,
                         hs);
  st = split_produce(s, q, k, v, scale, causal, runs, T, P, ws_m, ws_l, ws_acc, nullptr, nullptr,
                     hs);
  if (st != EF_OK) return st;
  ef::CombineParams c{};
  c.m = ws_m;
  c.l = ws_l;
  c.acc = ws_acc;
  c.o = o;
  c.rows = (int)s.rows();
  c.P = P;
  c.D = s.D;
  return from_hip(ef::launch_combine(c, hs));
}

}  // namespace

namespace ef {

// ef_attention_splitkv over a caller-chosen workspace, for the library's other
// entry points (the allocation-free variant passes its static scratch).
ef_status splitkv_into(const void* q, const void* k, const void* v, float* o, int B, int Hq,
                       int Hkv, int Sq, int Skv, int D, float scale, int causal,
                       int partition_size, void* workspace, size_t workspace_bytes,
                       void* stream) {
  return splitkv_impl(Shape{B, Hq, Hkv, Sq, Skv, D}, q, k, v, o, scale, causal,
                      key_runs(Sq, Skv, 0, 0), partition_size, workspace, workspace_bytes,
                      stream);
}

}  // namespace ef

extern "C" {

ef_status ef_attention_splitkv_partials(const void* q, const void* k, const void* v, int B,
                                        int Hq, int Hkv, int Sq, int Skv, int D, float scale,
                                        int causal, int partition_size, void* workspace,
                                        size_t workspace_bytes, void* stream) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  int T = 0, P = 0;
  float *ws_m = nullptr, *ws_l = nullptr, *ws_acc = nullptr;
  unsigned* counters = nullptr;
  // The output pointer is not used here; pass q so the shared check sees a non-null pointer.
  const ef::KeyRuns runs = key_runs(Sq, Skv, 0, 0);
  ef_status st = split_prepare(s, q, k, v, static_cast<const float*>(q), scale, runs,
                               partition_size, workspace, workspace_bytes, &T, &P, &ws_m, &ws_l,
                               &ws_acc, &counters);
  if (st != EF_OK || P == 0) return st;
  return split_produce(s, q, k, v, scale, causal, runs, T, P, ws_m, ws_l, ws_acc, nullptr,
                       nullptr, static_cast<hipStream_t>(stream));
}

ef_status ef_attention_splitkv(const void* q, const void* k, const void* v, float* o, int B,
                               int Hq, int Hkv, int Sq, int Skv, int D, float scale, int causal,
                               int partition_size, void* workspace, size_t workspace_bytes,
                               void* stream) {
  return splitkv_impl(Shape{B, Hq, Hkv, Sq, Skv, D}, q, k, v, o, scale, causal,
                      key_runs(Sq, Skv, 0, 0), partition_size, workspace, workspace_bytes,
                      stream);
}

ef_status ef_attention_splitkv_local(const void* q, const void* k, const void* v, float* o,
                                     int B, int Hq, int Hkv, int Sq, int Skv, int D, float scale,
                                     int window, int sinks, int partition_size, void* workspace,
                                     size_t workspace_bytes, void* stream) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  ef_status st = check_shape(s);
  if (st != EF_OK) return st;
  st = check_mask(window, sinks);
  if (st != EF_OK) return st;
  return splitkv_impl(s, q, k, v, o, scale, 1, key_runs(Sq, Skv, window, sinks), partition_size,
                      workspace, workspace_bytes, stream);
}

ef_status ef_attention_combine(const float* m, const float* l, const float* acc, float* o,
                               int rows, int num_partitions, int D, void* stream) {
  if (rows < 0 || num_partitions < 1) return EF_ERR_INVALID_SHAPE;
  if (D != 64 && D != 128) return EF_ERR_UNSUPPORTED_HEAD_DIM;
  if (rows == 0) return EF_OK;
  if (m == nullptr || l == nullptr || acc == nullptr || o == nullptr) return EF_ERR_NULL_POINTER;
  if (misaligned(m) || misaligned(l) || misaligned(acc) || misaligned(o)) return EF_ERR_MISALIGNED;
  ef::CombineParams c{};
  c.m = m;
  c.l = l;
  c.acc = acc;
  c.o = o;
  c.rows = rows;
  c.P = num_partitions;
  c.D = D;
  return from_hip(ef::launch_combine(c, static_cast<hipStream_t>(stream)));
}

double ef_attention_splitkv_modeled_us(int B, int Hq, int Hkv, int Sq, int Skv, int D, int window,
                                        int sinks, int partition_size) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  if (check_shape(s) != EF_OK || window < 0 || sinks < 0) return -1.0;
  if (partition_size <= 0 || partition_size % kTileKeys != 0) return -1.0;
  const ef::KeyRuns runs = key_runs(Sq, Skv, window, sinks);
  if (s.rows() == 0 || runs.lv == 0) return 0.0;
  return split_model_us(s, runs.lv, partition_size, visible_keys(s, runs));
}

int ef_attention_rows_per_workgroup(int B, int Hq, int Hkv, int Sq, int Skv, int D, int keys) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  if (check_shape(s) != EF_OK || keys < 0) return 0;
  return rows_per_block(s, keys);
}

int ef_attention_fwd_schedule(int B, int Hq, int Hkv, int Sq, int Skv, int D, int causal,
                              int window, int sinks) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  if (check_shape(s) != EF_OK || window < 0 || sinks < 0) return 0;
  if (s.rows() == 0 || Skv == 0) return 0;
  const FwdSchedule f =
      fwd_schedule(s, key_runs(Sq, Skv, window, sinks), causal != 0 || window > 0 ? 1 : 0);
  return f.bm + (f.key_split ? EF_SCHEDULE_KEY_SPLIT : 0) +
         (f.interleave ? EF_SCHEDULE_LONGEST_FIRST : 0);
}

ef_status ef_attention_splitkv_tune(const void* q, const void* k, const void* v, float* o, int B,
                                    int Hq, int Hkv, int Sq, int Skv, int D, float scale,
                                    int causal, int window, int sinks, void* workspace,
                                    size_t workspace_bytes, void* stream, int* partition_size) {
  if (partition_size == nullptr) return EF_ERR_NULL_POINTER;
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  ef_status st = check_shape(s);
  if (st != EF_OK) return st;
  if (window < 0 || sinks < 0 || (window == 0 && sinks != 0)) return EF_ERR_INVALID_MASK;
  st = check_io(s, q, k, v, o, scale);
  if (st != EF_OK) return st;
  const bool local = window > 0;
  const ef::KeyRuns runs = key_runs(Sq, Skv, window, sinks);
  if (s.rows() == 0 || runs.lv == 0) {
    *partition_size = resolve_partition(s, runs.lv, 0, visible_keys(s, runs));
    return EF_OK;
  }
  // Candidates the model rates best, whose workspace fits.
  std::vector<std::pair<double, int>> ranked;
  for (int t : partition_candidates(runs.lv)) {
    if (workspace_size_impl(s, runs, t) <= workspace_bytes)
      ranked.push_back({split_model_us(s, runs.lv, t, visible_keys(s, runs)), t});
  }
  if (ranked.empty()) return EF_ERR_WORKSPACE_TOO_SMALL;
  std::sort(ranked.begin(), ranked.end());
  constexpr size_t kTried = 6;
  if (ranked.size() > kTried) ranked.resize(kTried);
  std::vector<int> cands;
  for (const auto& r : ranked) cands.push_back(r.second);

  hipStream_t hs = static_cast<hipStream_t>(stream);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    return EF_ERR_HIP;
  }
  auto call = [&](int t) {
    return splitkv_impl(s, q, k, v, o, scale, local ? 1 : causal, runs, t, workspace,
                        workspace_bytes, stream);
  };
  // Successive halving (section 6.3, progressive tuning): time every
  // remaining candidate, keep the faster half, double the repetitions.
  int reps = 2;
  while (cands.size() > 1 && st == EF_OK) {
    std::vector<std::pair<float, int>> timed;
    for (int t : cands) {
      st = call(t);  // warm-up
      if (st != EF_OK) break;
      if (hipEventRecord(e0, hs) != hipSuccess) { st = EF_ERR_HIP; break; }
      for (int r = 0; r < reps && st == EF_OK; ++r) st = call(t);
      if (st != EF_OK) break;
      float ms = 0.f;
      if (hipEventRecord(e1, hs) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
          hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
        st = EF_ERR_HIP;
        break;
      }
      timed.push_back({ms, t});
    }
    if (st != EF_OK) break;
    std::stable_sort(timed.begin(), timed.end());
    cands.clear();
    for (size_t i = 0; i < (timed.size() + 1) / 2; ++i) cands.push_back(timed[i].second);
    reps *= 2;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (st == EF_OK) *partition_size = cands.front();
  return st;
}

}  // extern "C"

namespace {

// Row tiles of 128 rows from which a differential layer left to the library may
// run as one launch over both branches (a workgroup of eight waves per tile and
// CU) where the model would split: from about three quarters of the chip's CUs
// on, the second producer, the two combines and the stored states can cost more
// than the idle CUs. Measured below the line, split / one launch (us): 512 of
// 16384 keys, 128 tiles 290 / 411.
constexpr long long kDiffPairTiles = 192;

// Largest partition whose references one launch in its place renews.
constexpr int kRenewKeys = 8192;

// Times of the two ways from that line on (us). One launch runs ceil(tiles / 256)
// rounds of one workgroup per CU over the keys a row sees: 30 ns a key with every
// CU at work (18.3 at D = 64), 23 (16) with few, since the clock rises. The split's
// two producers share the work evenly but for the idle part of their last round
// and, under a causal mask with about as many queries as keys, partitions that end
// early; the partition states go through HBM twice, at 5.5 TB/s. Split / one launch
// measured (us): 1024 causal queries of 8192, 17472 and 65536 keys, row tiles in
// brackets, D = 128 [192] 236 / 206, 479 / 453, 1528 / 1672; [256] 273 / 244, 636 /
// 531, 2020 / 1973; [272] 346 / 417, 701 / 900, 2338 / 3700; [384] 437 / 433, -, 3031
// / 3718; [640] 734 / 677, 1599 / 1441, 4936 / 5866; D = 64 [192] 157 / 142, 271 / 296,
// 871 / 1094; [256] 176 / 153, 362 / 321, 1254 / 1226; [272] 205 / 279, 392 / 593, 1356
// / 2409; 9 heads of 128, 4096 of 4096 keys [288] causal 160 / 128, full 219 / 231.
// Over 150 such points, 192 to 1024 tiles of 2048 to 65536 keys, the pick was the
// faster way or within 2.3% of it.
constexpr double kDiffKeyUs128 = 30.0e-3, kDiffKeyUs64 = 18.3e-3;
constexpr double kDiffLoneKeyUs128 = 23.0e-3, kDiffLoneKeyUs64 = 16.0e-3;
constexpr double kDiffRenewCost = 1.015;       // renewals of the reference
constexpr double kDiffSplitKeyUs64 = 17.0e-3;  // at D = 128 as in one launch
constexpr double kDiffSplitIdle = 0.5;         // part of the last round's idle share that shows
constexpr double kDiffSplitCausal = 0.4;
constexpr double kDiffStateBytesPerUs = 5.5e6;
constexpr double kDiffSplitUs = 18.0;  // three more launches

bool diff_one_launch_faster(const Shape& s, int T, int causal) {
  const double R = (double)(s.Hq / s.Hkv) * s.Sq;
  const double rounds = (double)s.B * s.Hkv * std::ceil(R / 128.0) / 256.0;
  const double keys = s.Skv, queries = s.Sq, P = std::ceil(keys / T);
  double mean = keys, early = 0.0;  // keys a row sees; queries per key of a causal mask
  if (causal) {
    mean = queries <= keys ? keys - queries / 2 : keys * keys / (2 * queries);
    early = std::min(1.0, queries / keys);
  }
  const double key_us = s.D == 128 ? kDiffKeyUs128 : kDiffKeyUs64;
  const double lone_us = s.D == 128 ? kDiffLoneKeyUs128 : kDiffLoneKeyUs64;
  const double whole = std::floor(rounds), rest = rounds - whole;
  const double last = rest > 0 ? lone_us + (key_us - lone_us) * rest * rest * rest : 0.0;
  const double one = std::max((whole * key_us + last) * mean, lone_us * keys) *
                     (T <= kRenewKeys ? kDiffRenewCost : 1.0);
  const double split_key_us = s.D == 128 ? kDiffKeyUs128 : kDiffSplitKeyUs64;
  const double idle = kDiffSplitIdle * (std::ceil(rounds * P) / (rounds * P) - 1.0);
  const double work = 1.0 + idle + kDiffSplitCausal * early * early;
  const double split = rounds * split_key_us * mean * work +
                       4.0 * s.rows() * P * (s.D + 2) * 4.0 / kDiffStateBytesPerUs + kDiffSplitUs;
  return one <= split;
}

// And on short key axes, where two producers and two combines cost more than one
// workgroup's chain of tiles, whatever the grid. Measured, split / one launch
// (us): 6 x 4 heads of 128, 72 rows, 512 keys 25.0 / 21.0, 640 25.3 / 24.1, 1024
// 27.9 / 32.5; 4 x 12 heads of 64, 128 rows, 640 keys 24.9 / 18.3, 1024 27.8 /
// 24.4; 4 heads of 64, 64 rows, 640 keys 16.4 / 12.9, 1024 17.1 / 17.4; one row,
// 32 heads of 128, 256 keys 11.4 / 10.7, 512 13.8 / 16.0.
int diff_pair_keys(int D, long long R) {
  return R <= kDecodeMaxRows ? 256 : D == 64 ? 896 : 640;
}

// Whether the library may run this layer in one launch without being asked for
// one partition.
bool diff_pair_grid(const Shape& s) {
  const long long R = (long long)(s.Hq / s.Hkv) * s.Sq;
  return R > 64 && (long long)s.B * s.Hkv * ((R + 127) / 128) >= kDiffPairTiles;
}

// Number of partitions ef_diff_attention uses (1 = single pass), or 0 for an
// invalid shape or partition size. *T_out: keys per partition of the caller's or
// the model's split, also where one launch takes its place.
long long diff_partitions(const Shape& s, int partition_size, int causal, int* T_out) {
  if (check_shape(s) != EF_OK) return 0;
  if (partition_size < 0 || partition_size % kTileKeys != 0) return 0;
  if (s.rows() == 0 || s.Skv == 0) return 1;
  const long long R = (long long)(s.Hq / s.Hkv) * s.Sq;
  const int T = resolve_partition(s, s.Skv, partition_size, s.Skv);
  *T_out = T;
  if (partition_size == 0 && (s.Skv <= diff_pair_keys(s.D, R) ||
                              (diff_pair_grid(s) && diff_one_launch_faster(s, T, causal))))
    return 1;
  return (s.Skv + (long long)T - 1) / T;
}

// One branch through the split-KV producer and the combine; with `diff` the
// combine applies the differential epilogue against the A2 already in o.
ef_status diff_branch_split(const Shape& s, const void* q, const void* k, const void* v, float* o,
                            float scale, int causal, const ef::KeyRuns& runs, int T, int P,
                            const WsLayout& w, char* ws, const ef::DiffParams* diff,
                            hipStream_t hs) {
  float* ws_m = reinterpret_cast<float*>(ws + w.m_off);
  float* ws_l = reinterpret_cast<float*>(ws + w.l_off);
  float* ws_acc = reinterpret_cast<float*>(ws + w.acc_off);
  ef_status st = split_produce(s, q, k, v, scale, causal, runs, T, P, ws_m, ws_l, ws_acc, nullptr,
                               nullptr, hs);
  if (st != EF_OK) return st;
  ef::CombineParams c{};
  c.m = ws_m;
  c.l = ws_l;
  c.acc = ws_acc;
  c.o = o;
  c.rows = (int)s.rows();
  c.P = P;
  c.D = s.D;
  if (diff != nullptr) c.diff = *diff;
  return from_hip(ef::launch_combine(c, hs));
}

}  // namespace

extern "C" {

ef_status ef_diff_attention(const void* q1, const void* q2, const void* k1, const void* k2,
                            const void* v, float* o, const float* lambda_q1,
                            const float* lambda_k1, const float* lambda_q2,
                            const float* lambda_k2, const float* norm_weight, float lambda_init,
                            float eps, int B, int Hq, int Hkv, int Sq, int Skv, int D,
                            float scale, int causal, int partition_size, void* workspace,
                            size_t workspace_bytes, void* stream) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  ef_status st = check_shape(s);
  if (st != EF_OK) return st;
  if (partition_size < 0 || partition_size % kTileKeys != 0) return EF_ERR_INVALID_PARTITION;
  st = check_io(s, q1, k1, v, o, scale);
  if (st != EF_OK) return st;
  st = check_io(s, q2, k2, v, o, scale);
  if (st != EF_OK) return st;
  if (!std::isfinite(lambda_init) || !std::isfinite(eps) || eps < 0.f) return EF_ERR_INVALID_DIFF;
  if (s.rows() == 0) return EF_OK;
  if (lambda_q1 == nullptr || lambda_k1 == nullptr || lambda_q2 == nullptr ||
      lambda_k2 == nullptr || norm_weight == nullptr)
    return EF_ERR_NULL_POINTER;
  if (misaligned(norm_weight)) return EF_ERR_MISALIGNED;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  // No keys: A1 = A2 = 0, so y = 0 and every output row is 0.
  if (s.Skv == 0) return from_hip(ef::launch_zero_fill(o, (size_t)s.rows() * s.D, hs));
  int T = 0;
  long long P = diff_partitions(s, partition_size, causal, &T);
  if (P > kMaxGridYZ) return EF_ERR_INVALID_PARTITION;
  // Large grids left to the library do without a workspace: they run in one launch,
  // if slower.
  const WsLayout w = ws_layout(s.rows(), P, s.D);
  if (partition_size == 0 && diff_pair_grid(s) &&
      (workspace == nullptr || workspace_bytes < w.bytes || misaligned(workspace)))
    P = 1;
  const ef::DiffParams diff{lambda_q1, lambda_k1, lambda_q2, lambda_k2, norm_weight, lambda_init,
                            eps};
  const ef::KeyRuns runs = key_runs(Sq, Skv, 0, 0);
  if (P == 1) {
    // Where one launch takes the place of a split, a row's reference is renewed as
    // often as the split's partitions would have set one of their own: each sets
    // its largest weight to exactly 1, free of the rounding to bf16. Without the
    // renewal the error against 64 bits was 23% above the split's with ten 64-key
    // partitions (640 keys: 2.06e-3, split 1.66e-3), 0.5% with five of 2048, 0.2%
    // with two of 4096. With partitions of 16384 keys the two agree (-0.2% to 0.1%
    // over eight pairs of inputs), and the plain form is 1.2% faster (32 heads of
    // 128, 1024 of 32768 keys 1020 / 1008 us).
    const int renew = T < Skv && T <= kRenewKeys ? T / kTileKeys : 0;
    return launch_mfma(s, q1, k1, v, o, nullptr, nullptr, nullptr, runs.lv, 1, scale, causal,
                       runs, hs, q2, k2, &diff, renew);
  }
  if (workspace == nullptr || workspace_bytes < w.bytes) return EF_ERR_WORKSPACE_TOO_SMALL;
  if (misaligned(workspace)) return EF_ERR_MISALIGNED;
  char* ws = static_cast<char*>(workspace);
  st = diff_branch_split(s, q2, k2, v, o, scale, causal, runs, T, (int)P, w, ws, nullptr, hs);
  if (st != EF_OK) return st;
  return diff_branch_split(s, q1, k1, v, o, scale, causal, runs, T, (int)P, w, ws, &diff, hs);
}

size_t ef_diff_attention_workspace_size(int B, int Hq, int Hkv, int Sq, int Skv, int D,
                                        int partition_size) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  int T = 0;
  const long long P = std::max(diff_partitions(s, partition_size, 0, &T),
                               diff_partitions(s, partition_size, 1, &T));
  if (P <= 1 || P > kMaxGridYZ) return 0;
  return ws_layout(s.rows(), P, s.D).bytes;
}

}  // extern "C"

namespace {

// Partitions of the output-channel split decode (1: no workspace), or 0 for an
// invalid shape, partition size or split.
long long dsplit_partitions(const Shape& s, int d_splits, int partition_size, int* T_out) {
  if (check_shape(s) != EF_OK) return 0;
  if (d_splits != 1 && d_splits != 2 && d_splits != 4) return 0;
  if ((long long)(s.Hq / s.Hkv) * s.Sq > kDecodeMaxRows) return 0;
  if (partition_size < 0 || partition_size % kTileKeys != 0) return 0;
  if (s.rows() == 0 || s.Skv == 0) return 1;
  const int T = resolve_partition(s, s.Skv, partition_size, s.Skv);
  *T_out = T;
  return (s.Skv + (long long)T - 1) / T;
}

}  // namespace

extern "C" {

ef_status ef_attention_decode_dsplit(const void* q, const void* k, const void* v, float* o, int B,
                                     int Hq, int Hkv, int Sq, int Skv, int D, float scale,
                                     int causal, int d_splits, int partition_size,
                                     void* workspace, size_t workspace_bytes, void* stream) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  ef_status st = check_shape(s);
  if (st != EF_OK) return st;
  if (d_splits != 1 && d_splits != 2 && d_splits != 4) return EF_ERR_INVALID_SPLIT;
  if ((long long)(Hq / Hkv) * Sq > kDecodeMaxRows) return EF_ERR_INVALID_SPLIT;
  if (partition_size < 0 || partition_size % kTileKeys != 0) return EF_ERR_INVALID_PARTITION;
  st = check_io(s, q, k, v, o, scale);
  if (st != EF_OK) return st;
  if (s.rows() == 0) return EF_OK;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (s.Skv == 0) return from_hip(ef::launch_zero_fill(o, (size_t)s.rows() * s.D, hs));
  int T = 0;
  const long long P = dsplit_partitions(s, d_splits, partition_size, &T);
  if (P < 1 || P * d_splits > 0x7fffffffLL) return EF_ERR_INVALID_PARTITION;
  const ef::KeyRuns runs = key_runs(Sq, Skv, 0, 0);
  if (P == 1)  // each workgroup writes its channels of o: no workspace, no merge
    return split_produce(s, q, k, v, scale, causal, runs, T, 1, nullptr, nullptr, nullptr,
                         nullptr, o, hs, d_splits);
  const WsLayout w = ws_layout(s.rows(), P, s.D);
  if (workspace == nullptr || workspace_bytes < w.bytes) return EF_ERR_WORKSPACE_TOO_SMALL;
  if (misaligned(workspace)) return EF_ERR_MISALIGNED;
  char* ws = static_cast<char*>(workspace);
  float* ws_m = reinterpret_cast<float*>(ws + w.m_off);
  float* ws_l = reinterpret_cast<float*>(ws + w.l_off);
  float* ws_acc = reinterpret_cast<float*>(ws + w.acc_off);
  unsigned* counters = reinterpret_cast<unsigned*>(ws + w.cnt_off);
  if (fused_combine(s, P, d_splits))
    return split_produce(s, q, k, v, scale, causal, runs, T, (int)P, ws_m, ws_l, ws_acc,
                         counters, o, hs, d_splits);
  st = split_produce(s, q, k, v, scale, causal, runs, T, (int)P, ws_m, ws_l, ws_acc, nullptr,
                     nullptr, hs, d_splits);
  if (st != EF_OK) return st;
  ef::CombineParams c{};
  c.m = ws_m;
  c.l = ws_l;
  c.acc = ws_acc;
  c.o = o;
  c.rows = (int)s.rows();
  c.P = (int)P;
  c.D = s.D;
  return from_hip(ef::launch_combine(c, hs));
}

size_t ef_attention_decode_dsplit_workspace_size(int B, int Hq, int Hkv, int Sq, int Skv, int D,
                                                 int d_splits, int partition_size) {
  const Shape s{B, Hq, Hkv, Sq, Skv, D};
  int T = 0;
  const long long P = dsplit_partitions(s, d_splits, partition_size, &T);
  if (P <= 1) return 0;
  return ws_layout(s.rows(), P, s.D).bytes;
}

}  // extern "C"
