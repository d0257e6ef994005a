// Tiled rolling attention on bf16 MFMA (form M2 of figure
// "attention-rewrites", section 3; code-generation mapping of section 6.1:
// the query-row tile axis is the grid, the key-tile axis is the loop inside a
// workgroup, and the (max, sum, value) reducer state is loop-carried).
//
// A workgroup holds NW waves and 32*NW query rows of one kv head. Rows are
// packed as r = sq*G + g, so the Hq/Hkv query heads that read the same kv
// head share every K/V tile the workgroup stages (replication by index,
// section 3.1). Each wave owns 32 rows and works on transposed tiles:
//
//   S^T[key][query] = K_tile (A operand, from LDS) * Q^T (B operand, registers)
//   O^T[d][query]  += V^T_tile (A operand, from LDS) * P^T (B operand, registers)
//
// with v_mfma_f32_32x32x16_bf16. In both products lane l owns query l % 32,
// so the row max, the exponentials, the row sum and the rescale of the
// carried value are lane-local, and the score accumulator, converted to bf16,
// is already in the B-operand layout of the second product. Two lanes
// (l and l ^ 32) share a query and exchange one value per tile for the max.
//
// Two loops share this layout and the prologue and epilogue around it:
//
// The rolling loop (struct Rolling; prefill and every launch whose K/V tiles
// are shared or whose rows fill the matrix core) works on 32-key subtiles of
// 64-key tiles. While the vector ALU turns subtile j's scores into weights, the
// matrix core forms subtile j + 1's scores and multiplies subtile j - 1's
// values: three subtiles are in flight, so nothing the wave issues during a
// subtile waits for another kind of its work, and the source fixes the order of
// issue product by product (see struct Rolling). K is staged one tile ahead of
// V, two stages each, one workgroup barrier per 64 keys.
//
// The streaming loop (pipelined_step; the split producer of decode shapes)
// works on 32-key tiles of half the LDS, four workgroups to a compute unit,
// with non-temporal loads: it is bound by the K/V stream. Tile j's weights are
// formed while the matrix core computes tile j + 1's scores, then tile j's
// values are multiplied.
//
// Tiles go from HBM straight into LDS (direct loads, no staging registers),
// row-major with their 16-byte chunks permuted per row so that the fragment
// reads are free of bank conflicts. The V^T operand of the second product comes
// from transposing LDS reads (ds_read_b64_tr_b16) of the row-major V tile, in
// the key order of the P^T fragments.
//
// The exponent reference is only moved up when a weight against it may exceed
// 2^8 (base-2 units), so the carried sum and value are rescaled rarely; the
// final value / sum is unchanged (the repair h(c, s, s') = c * 2^(s - s') is
// exact for any reference point). A negative scale is moved into q (bf16
// negation is exact), so the scale c below is positive.
//
// In split mode the workgroup covers one key partition and stores the
// partition's (reference, sum, value) state instead of value / sum.
//
// Local attention (a causal sliding window of W keys plus S sink keys; the
// sliding-window GQA and attention-sink layers of section 7.3) visits only
// the tiles some row of the workgroup can see: the tiles of the sink run
// [0, S) and those from the window start of the workgroup's first row to its
// causal end. Both runs feed the same rolling reducer, so the sink and window
// keys share one softmax normalisation; the keys in between are never read.
//
// Differential attention (section 7.3), single pass: one launch, two groups of
// waves, one per branch. They meet in LDS, form y = A1 - lambda * A2, mix in
// lambda from the four learned vectors, RMS-normalise the row over D and write
// the result, so neither branch's output reaches HBM.
#include "diff_norm.hpp"
#include "ef_device.hpp"
#include "ef_kernels.hpp"

namespace ef {

namespace {

constexpr float kLazyThreshold = 8.f;  // base-2 headroom before the reference moves
constexpr float kLazySum = 256.f;      // 2^8: a lane's weights whose sum is below are too
constexpr float kNoRef = -3.402823466e+38f;  // rolling loop: no key seen yet (-FLT_MAX)
constexpr float kRenewDepth = 16.f;  // a renewed reference lies at most this far below the top

// Geometry of K and V rows in LDS.
template <int D>
struct TileGeom {
  static constexpr int KCH = D / 8;        // 16-byte chunks per row
  static constexpr int ROW = 2 * D;        // bytes per K or V row (no padding: swizzled)
  static constexpr int RPI = 64 / KCH;     // rows one wave-wide direct load fills (1 KiB)
  static constexpr int SUB = 32 * ROW;     // bytes of 32 rows
  // Streaming loop: V stage 0, V stage 1, K stage 0, K stage 1 of 32 keys each.
  template <int S>
  static constexpr int v_off() { return S * SUB; }
  template <int S>
  static constexpr int k_off() { return (2 + S) * SUB; }
  // Tiles sit row-major in LDS with their 16-byte chunks permuted per row
  // (chunk c of row r at slot c ^ swz(r)), so the fragment reads below hit
  // distinct banks: K rows are read 16 rows at a time at one chunk, V rows four
  // rows at a time at 32 consecutive bytes (transposing reads).
  static __device__ __forceinline__ int swz_k(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
  static __device__ __forceinline__ int swz_v(int r) {
    return D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1);
  }
};

// Cross-half exchange: max of x over lanes l and l ^ 32.
__device__ __forceinline__ float max_with_other_half(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Key tiles of one workgroup, in visiting order: `na` tiles of the sink run
// starting at key a0 (keys below aend), then the tiles of the window run
// starting at b0 (keys below bend). Without a window the sink run is empty and
// the window run is the whole key range. Tiles past the last one cover no key.
template <int BN>
struct TileList {
  int a0, aend, na, b0, bend, n;
  int full_lo;  // a tile whose last key is at most this is below every row's causal limit
  int win_lo;   // a tile starting at or above this key lies in every row's window
  int sinks;    // keys below this are visible whatever the window
  __device__ __forceinline__ int base(int j) const {
    return j < na ? a0 + j * BN : b0 + (j - na) * BN;
  }
  __device__ __forceinline__ int end(int j) const { return j < na ? aend : bend; }
  // Whether some key of tile j is hidden from some row of the workgroup.
  __device__ __forceinline__ bool masked(int j) const {
    const int kb = base(j);
    return kb + BN > end(j) || kb + BN - 1 > full_lo || (kb < win_lo && kb + BN > sinks);
  }
};

// Loads of the streaming loop's 32-key tiles, straight from HBM to LDS (one
// 16-byte chunk per lane and load, each wave-wide load filling RPI whole rows).
// Rows past the tile's run repeat its last row (their keys are masked, their
// values finite); a tile past the last one loads nothing. Every key is read
// exactly once, so the loads are non-temporal and stream past the caches, which
// lifts the read rate by about a sixth (5.5 to 6.3-6.5 TB/s on the 537 MB of a
// 16 x 8192-key chunked decode).
template <int D, int NW>
struct Loader {
  using G = TileGeom<D>;
  static constexpr int INSTS = 32 / G::RPI / NW;  // direct loads per wave and tile
  static_assert(INSTS * G::RPI * NW == 32, "tile split over the waves");
  int row[INSTS];       // tile row whose chunk this lane loads
  int kchunk[INSTS];    // element offset of that chunk in a K row
  int vchunk[INSTS];    // element offset of that chunk in a V row
  unsigned koff[INSTS];  // byte offset of this lane's K chunk from the tile's first row
  unsigned voff[INSTS];  // the same for V
  int wave;              // wave index, uniform (scalar)

  __device__ __forceinline__ void init() {
    const int lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int i = 0; i < INSTS; ++i) {
      const int blk = wave + NW * i;
      row[i] = blk * G::RPI + lane / G::KCH;
      const int slot = lane % G::KCH;
      kchunk[i] = (slot ^ G::swz_k(row[i])) * 8;
      vchunk[i] = (slot ^ G::swz_v(row[i])) * 8;
      koff[i] = (unsigned)(row[i] * D + kchunk[i]) * 2u;
      voff[i] = (unsigned)(row[i] * D + vchunk[i]) * 2u;
    }
  }

  static __device__ __forceinline__ void load_chunk(const char* g, char* l) {
    __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void*)l, 16, 0,
                                     2 /* non-temporal */);
  }
  // The address is a uniform base (the tile's first row) plus a 32-bit lane
  // offset, so the vector ALU only clamps rows of a ragged tile.
  template <bool ISK>
  __device__ __forceinline__ void load(char* stage, const uint16_t* head, int kb, int kend) const {
    const int nrows = kend - kb;
    if (nrows <= 0) return;
    const char* base = reinterpret_cast<const char*>(head + (size_t)kb * D);
    if (nrows >= 32) {
#pragma unroll
      for (int i = 0; i < INSTS; ++i)
        load_chunk(base + (ISK ? koff[i] : voff[i]), stage + (wave + NW * i) * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < INSTS; ++i) {
        const int r = min(row[i], nrows - 1);
        const unsigned off = (unsigned)(r * D + (ISK ? kchunk[i] : vchunk[i])) * 2u;
        load_chunk(base + off, stage + (wave + NW * i) * 1024);
      }
    }
  }
  template <int S>
  __device__ __forceinline__ void load_k(char* smem, const uint16_t* kh, int kb, int kend) const {
    load<true>(smem + G::template k_off<S>(), kh, kb, kend);
  }
  template <int S>
  __device__ __forceinline__ void load_v(char* smem, const uint16_t* vh, int kb, int kend) const {
    load<false>(smem + G::template v_off<S>(), vh, kb, kend);
  }
};

// Waits for this wave's direct-to-LDS loads (they count as vector memory loads).
__device__ __forceinline__ void wait_tile_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }

// Scores of the keys hidden from this lane's row set to -inf: past the run's end
// or the causal limit `lim`, or at most `lo` (left of the window) and not a sink.
// Element i holds key kb + 4 h + o(i) with a compile-time offset o, so the hidden
// keys become per-lane offset thresholds, clamped to the tile so the arithmetic
// cannot overflow: past `vis`, and inside [wlo, whi]. Selects, not branches.
__device__ __forceinline__ void mask_scores(floatx16& x, int kb, int kend, int lim, int lo,
                                            int sinks, int h) {
  const int base = kb + 4 * h;
  const int vis = min(min(kend - 1, lim), kb + 32) - base;
  const int wlo = max(sinks, kb) - base;
  const int whi = min(max(lo, kb - 1), kb + 32) - base;
  if (__builtin_amdgcn_ballot_w64(whi >= wlo)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int o = 8 * (i >> 2) + (i & 3);
      const bool hide = (o > vis) | ((o >= wlo) & (o <= whi));
      x[i] = hide ? kNegInf : x[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int o = 8 * (i >> 2) + (i & 3);
      x[i] = o > vis ? kNegInf : x[i];
    }
  }
}

// S^T of the 32-key subtile at kt, every K fragment in registers of its own so
// that the reads run several products ahead.
template <int D>
__device__ __forceinline__ void subtile_scores(const char* kt, const int* kread,
                                               const bf16x8_t* qf, floatx16& sacc) {
  u32x4_t kx[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) kx[s] = *reinterpret_cast<const u32x4_t*>(kt + kread[s]);
#pragma unroll
  for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, kx[s]), qf[s],
                                                   sacc, 0, 0, 0);
}

// S^T of both 32-key subtiles of the 64-key tile at kt, their products alternating.
template <int D>
__device__ __forceinline__ void tile_scores(const char* kt, const int* kread, const bf16x8_t* qf,
                                            floatx16& x0, floatx16& x1) {
  constexpr int SUB = TileGeom<D>::SUB;
#pragma unroll
  for (int i = 0; i < 16; ++i) x0[i] = x1[i] = 0.f;
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    const u32x4_t k0 = *reinterpret_cast<const u32x4_t*>(kt + kread[s]);
    const u32x4_t k1 = *reinterpret_cast<const u32x4_t*>(kt + SUB + kread[s]);
    x0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, k0), qf[s], x0, 0,
                                                0, 0);
    x1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, k1), qf[s], x1, 0,
                                                0, 0);
  }
}

// Softmax and value steps of the streaming loop's 32-key tiles.
template <int D>
struct Tile {
  using Geo = TileGeom<D>;
  static constexpr int DT = D / 32;  // 32-wide output tiles along D

  // Masks the scores and updates the rolling reference; returns -reference (0
  // while nothing is visible).
  static __device__ __forceinline__ float prepare(floatx16& x, floatx16* oacc, float& lsum,
                                                  float& mref, float c, int kb, int kend,
                                                  bool masked, int lim, int lo, int sinks,
                                                  int h) {
    if (masked) mask_scores(x, kb, kend, lim, lo, sinks, h);
    float tmax = fmaxf(x[0], x[1]);
#pragma unroll
    for (int i = 2; i < 16; ++i) tmax = fmaxf(tmax, x[i]);
    tmax = max_with_other_half(tmax);
    const float cand = tmax * c;  // tile maximum in base-2 units (c > 0)
    // Move the reference only when the tile exceeds it by the threshold.
    const bool up = cand > mref + kLazyThreshold;
    if (__builtin_amdgcn_ballot_w64(up)) {
      const float rs = up ? exp2_fast(mref - cand) : 1.f;  // 0 when mref = -inf
      mref = up ? cand : mref;
      lsum *= rs;
#pragma unroll
      for (int i = 0; i < DT; ++i)
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) oacc[i][jj] *= rs;
    }
    return (mref == kNegInf) ? 0.f : -mref;
  }

  // Weights 2^(x*c - reference) as bf16 pairs (P^T fragments) and their row
  // sum in fp32. (A packed bf16 dot product with (1, 1) per pair would sum the
  // rounded weights in half the instructions, but between matrix products it
  // costs about ten cycles each; the two sums differ by far less than the
  // rounding of the weights themselves.)
  static __device__ __forceinline__ void weights(const floatx16& x, float c, float mneg,
                                                 uint32_t* pk, float& lsum) {
    float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float p0 = exp2_fast(fmaf(x[2 * i], c, mneg));
      const float p1 = exp2_fast(fmaf(x[2 * i + 1], c, mneg));
      pk[i] = pack_bf16x2(p0, p1);
      ps[i & 3] += p0 + p1;
    }
    lsum += (ps[0] + ps[1]) + (ps[2] + ps[3]);
  }

  // O^T += V^T * P^T over the two 16-key steps of the tile in V stage S; the
  // V^T operand (8 keys of one value column per lane) comes from two transposing
  // reads of 4 keys each out of the row-major V tile. The reads are issued from
  // assembly: the compiler cannot tell them from the direct-to-LDS loads into the other
  // stages still in flight, and waits for every outstanding load before the
  // first of them, which leaves the step's loads only its first half to land.
  // The reads of 16-key step s + 1 are requested before the products of step
  // s; LDS operations complete in order, so before step s's products a wait
  // until at most step s + 1's reads are outstanding suffices (other
  // operations counted by the same counter only make it longer). An empty
  // statement that rewrites the operands after the wait keeps the products
  // below it.
  template <int S>
  static __device__ __forceinline__ void values(const char* smem, const int* vread,
                                                    const uint32_t* pk, floatx16* oacc) {
    constexpr int STEPS = 2;
    constexpr int READS = 2 * DT;  // reads per 16-key step
    static_assert(READS <= 15, "outstanding reads exceed the LDS counter");
    const unsigned base = (unsigned)(uintptr_t)(
        (const __attribute__((address_space(3))) char*)(smem + Geo::template v_off<S>()));
    u32x2_t lo[2][DT], hi[2][DT];
    auto read_step = [&](int s, u32x2_t(&l)[DT], u32x2_t(&h)[DT]) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const unsigned addr = base + vread[dt] + 16 * s * Geo::ROW;
        asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(l[dt]) : "v"(addr));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2"
                     : "=v"(h[dt])
                     : "v"(addr), "i"(8 * Geo::ROW));
      }
    };
    read_step(0, lo[0], hi[0]);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const int b = s & 1;
      if (s + 1 < STEPS) {
        read_step(s + 1, lo[b ^ 1], hi[b ^ 1]);
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"i"(READS) : "memory");
      } else {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) asm volatile("" : "+v"(lo[b][dt]), "+v"(hi[b][dt]));
      // P^T fragment: registers 8*(s%2) .. +8 of score half s/2, i.e. pk[4*s .. 4*s+3].
      const u32x4_t pv = {pk[4 * s], pk[4 * s + 1], pk[4 * s + 2], pk[4 * s + 3]};
      const bf16x8_t pf = __builtin_bit_cast(bf16x8_t, pv);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const u32x4_t vx = {lo[b][dt][0], lo[b][dt][1], hi[b][dt][0], hi[b][dt][1]};
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, vx), pf,
                                                          oacc[dt], 0, 0, 0);
      }
    }
  }
};

// One step of the streaming loop on tile j (stage parity S = j % 2). On entry
// sacc[S] holds S^T of tile j, K stage 1-S holds tile j+1 and V stage S holds
// tile j. The step requests K of tile j+2 (into K stage S, last read for tile j's
// scores) and V of tile j+1 (into V stage 1-S, last read for tile j-1's values)
// straight into LDS, computes tile j's weights while the matrix core computes
// tile j+1's scores, multiplies tile j's values, and waits for its loads before
// the workgroup barrier.
template <int D, int NW, int S>
__device__ __forceinline__ void pipelined_step(char* smem, const Loader<D, NW>& ld,
                                               const uint16_t* kh, const uint16_t* vh,
                                               const TileList<32>& tl, int j, int lim, int lo,
                                               int h, const int* kread, const int* vread,
                                               const bf16x8_t* qf, floatx16* sacc, floatx16* oacc,
                                               float& lsum, float& mref, float c) {
  using TileT = Tile<D>;
  ld.template load_k<S>(smem, kh, tl.base(j + 2), tl.end(j + 2));  // nothing past the last tile
  ld.template load_v<1 - S>(smem, vh, tl.base(j + 1), tl.end(j + 1));
  const float mneg = TileT::prepare(sacc[S], oacc, lsum, mref, c, tl.base(j), tl.end(j),
                                    tl.masked(j), lim, lo, tl.sinks, h);
  uint32_t pk[8];
  TileT::weights(sacc[S], c, mneg, pk, lsum);
  // Tile j+1's scores go to the other accumulator, so tile j's stay in place.
  subtile_scores<D>(smem + TileGeom<D>::template k_off<1 - S>(), kread, qf, sacc[1 - S]);
  TileT::template values<S>(smem, vread, pk, oacc);
  // The wait stays behind the products: the scheduler moves it up into them, where
  // the loads have had two thirds of the step to land (8 rows per kv head, 8 x
  // 16384 keys of 64: 65.7 -> 61.3 us; 16 x 12 heads, 8 of 2000 keys of 128: 43.9 ->
  // 41.6 us).
  __builtin_amdgcn_sched_barrier(0);
  wait_tile_loads();
  __syncthreads();
}

// Compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>).
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// The rolling loop's work on one 32-key subtile j: its softmax, beside the
// scores of subtile j + 1 and the values of subtile j - 1.
//
// What bounds it: the matrix core and, on long launches, the power limit (the
// clock falls from 2.4 to about 1.75 GHz under this loop; a library matrix
// product of random bf16 data runs at 1.77 GHz too). Before, a step formed a
// tile's weights and multiplied its values one after the other, took the tile's
// maximum on every step and spent about a hundred scalar instructions on tile
// addresses; its matrix cores were busy 54% of the time on 8192 keys at
// D = 128, whatever order the compiler issued the step in. Here
//  - all products of a subtile are independent of the softmax beside them, and
//    scheduling barriers pin one product, its share of the vector work (3-4
//    instructions) and the fragment reads PF products ahead to each slot;
//  - the maximum is only taken when a lane's sum of weights passes 2^8
//    (soft_end), 57 vector instructions per 16 weights instead of 74;
//  - tile loads keep one address register set for all tiles (StageLoader).
// Together the matrix cores are busy 61.5-63% of the time: 8192 x 8192 keys,
// 32/8 heads, 1064 -> 984 us; causal 4 x 2048, 168.5 -> 156.5 us; 1024 of 32768
// keys, 32 heads, one branch 521 -> 490 us. Tried on top, not kept: fragments
// read 4, 5 or 7 slots ahead (equal); eight waves sharing each tile (clock 1.89
// GHz but 59.6% busy: 8192^2 920 us against 945, causal 4 x 2048 160 against 154);
// 64 rows per wave, one wave per SIMD (half the fragment reads, 2.1 GHz, 51%
// busy: 952 and 171 us); three or four stages per tile (25 us against 20 on a
// 777-token prompt).
template <int D>
struct Rolling {
  using Geo = TileGeom<D>;
  static constexpr int KSTEPS = D / 16;
  static constexpr int DT = D / 32;
  static constexpr int NV = 2 * DT;            // value products of a subtile
  static constexpr int SLOTS = KSTEPS + NV;    // products of a subtile
  static constexpr int PF = 6;                 // slots a fragment is read ahead of its product

  // Products of a subtile in issue order: scores and values alternate, so that
  // a product rarely follows the one it accumulates onto. The last two are
  // values, so the scores are complete when the next subtile reads them; that
  // leaves the last two scores one behind the other, the subtile's one dependent
  // pair.
  static constexpr bool is_score(int i) {
    return i < SLOTS - 4 ? i % 2 == 0 : i < SLOTS - 2;
  }
  static constexpr int index_of(int i) {  // k-step of a score slot, number of a value slot
    int n = 0;
    for (int k = 0; k < i; ++k) n += is_score(k) == is_score(i);
    return n;
  }

  // Fragment offsets and operands of the wave, and the state carried along.
  const int* kread;
  const int* vread;
  const bf16x8_t* qf;
  floatx16* oacc;
  float& lsum;
  float& mref;
  float c;

  // Fragment of product i of a subtile, K and V subtiles at kt and vt.
  template <int I>
  __device__ __forceinline__ u32x4_t fragment(const char* kt, const char* vt) const {
    constexpr int n = index_of(I);
    if constexpr (is_score(I)) {
      return *reinterpret_cast<const u32x4_t*>(kt + kread[n]);
    } else {
      typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
      const char* p = vt + vread[n % DT] + 16 * (n / DT) * Geo::ROW;
      const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
          (__attribute__((address_space(3))) bf16x4_t*)(p));
      const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
          (__attribute__((address_space(3))) bf16x4_t*)(p + 8 * Geo::ROW));
      const bf16x8_t vx = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      return __builtin_bit_cast(u32x4_t, vx);
    }
  }

  template <int I>
  __device__ __forceinline__ void product(const u32x4_t& fr, floatx16& y, const uint32_t* pin) {
    constexpr int n = index_of(I);
    if constexpr (is_score(I)) {
      if constexpr (n == 0) {
        floatx16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
        y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fr), qf[0], z, 0,
                                                   0, 0);
      } else {
        y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fr), qf[n], y, 0,
                                                   0, 0);
      }
    } else {
      constexpr int s = n / DT, dt = n % DT;
      const u32x4_t pv = {pin[4 * s], pin[4 * s + 1], pin[4 * s + 2], pin[4 * s + 3]};
      oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          __builtin_bit_cast(bf16x8_t, fr), __builtin_bit_cast(bf16x8_t, pv), oacc[dt], 0, 0, 0);
    }
  }

  // One subtile's softmax (scores x, weights pout) beside the other subtiles'
  // products: slot I's share of the weights 2^(x c - reference) and their sum.
  struct Soft {
    float ps[4];
    float prev;
  };
  template <int I, int N>
  __device__ __forceinline__ void soft_slot(Soft& f, const floatx16& x, uint32_t* pout) const {
    constexpr int lo = 16 * I / N, hi = 16 * (I + 1) / N;
    static_for<hi - lo>([&](auto q) {
      constexpr int e = lo + decltype(q)::value;
      const float p = exp2_fast(fmaf(x[e], c, -mref));
      if constexpr (e % 2 == 0) {
        f.prev = p;
      } else {
        pout[e / 2] = pack_bf16x2(f.prev, p);
        if constexpr (e / 2 < 4)
          f.ps[e / 2] = f.prev + p;
        else
          f.ps[e / 2 - 4] += f.prev + p;
        // Keeps the weights' work in this slot (the compiler would sink it past
        // the branch of soft_end, next to its use).
        asm volatile("" : "+v"(pout[e / 2]), "+v"(f.ps[(e / 2) % 4]));
      }
    });
  }
  // The first tile's scores (x0, x1) set the reference to the row's maximum over
  // its 64 keys, and x0's weights are formed. Taken over the first subtile alone,
  // the reference was below more rows' largest score, whose weight then is no
  // longer exactly 1 but rounded to bf16: the error against 64 bits of 64 keys at
  // D = 64 was 1.50e-3 instead of 1.33e-3, of 384 keys 1.62e-3 instead of 1.60e-3.
  __device__ __forceinline__ void start(const floatx16& x0, const floatx16& x1, uint32_t* pout) {
    mref = fmaxf(mref, tile_max(x0, x1));
    Soft f;
    soft_slot<0, 1>(f, x0, pout);
    lsum += (f.ps[0] + f.ps[1]) + (f.ps[2] + f.ps[3]);
  }
  // A tile that renews the reference: it moves to the maximum of the tile, down as
  // well as up, and the carried sum and value move with it. Down at most
  // kRenewDepth below the largest so far (`top`), so that they grow by 2^kRenewDepth
  // at most; weights further below round to nothing that matters.
  __device__ __forceinline__ void renew(float& top, const floatx16& x0, const floatx16& x1,
                                        uint32_t* pout) {
    const float old = mref;
    top = fmaxf(top, old);
    mref = fmaxf(top - kRenewDepth, tile_max(x0, x1));  // kNoRef - kRenewDepth is kNoRef
    rescale(exp2_fast(old - mref));
    start(x0, x1, pout);
  }
  // Largest score of a row in a 64-key tile, base-2 units.
  __device__ __forceinline__ float tile_max(const floatx16& x0, const floatx16& x1) const {
    float tmax = fmaxf(x0[0], x1[0]);
#pragma unroll
    for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, fmaxf(x0[i], x1[i]));
    return max_with_other_half(tmax) * c;
  }
  // Moves the carried sum and value to another reference.
  __device__ __forceinline__ void rescale(float rs) {
    lsum *= rs;
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
      for (int jj = 0; jj < 16; ++jj) oacc[i][jj] *= rs;
  }
  // A lane's weights are all at most 2^8 when their sum is, and then the
  // reference stays. Otherwise (a row's first visible keys past its first tile, or
  // a larger score) the reference moves up to the subtile's maximum, the carried
  // sum and value are rescaled and the weights formed again.
  __device__ __forceinline__ void soft_end(Soft& f, const floatx16& x, uint32_t* pout) {
    float sum = (f.ps[0] + f.ps[1]) + (f.ps[2] + f.ps[3]);
    if (__builtin_amdgcn_ballot_w64(!(sum <= kLazySum))) {
      float tmax = fmaxf(x[0], x[1]);
#pragma unroll
      for (int i = 2; i < 16; ++i) tmax = fmaxf(tmax, x[i]);
      const float cand = max_with_other_half(tmax) * c;
      const float old = mref;
      mref = fmaxf(mref, cand);
      rescale(exp2_fast(old - mref));  // by 1 where the reference stayed
      soft_slot<0, 1>(f, x, pout);
      sum = (f.ps[0] + f.ps[1]) + (f.ps[2] + f.ps[3]);
    }
    lsum += sum;
  }

  // Subtile softmax of x into pout, the next subtile's scores into y (K subtile
  // at kt) and the values of the previous subtile (V subtile at vt, weights pin).
  // With CARRY_IN the first PF fragments are in carry, with CARRY_OUT the next
  // subtile's first PF are left there.
  template <bool CARRY_IN, bool CARRY_OUT>
  __device__ __forceinline__ void subtile(const floatx16& x, floatx16& y, const uint32_t* pin,
                                          uint32_t* pout, const char* kt, const char* vt,
                                          const char* kt2, const char* vt2, u32x4_t* carry) {
    u32x4_t fr[SLOTS];
    static_for<PF>([&](auto i) {
      constexpr int I = decltype(i)::value;
      if constexpr (CARRY_IN) fr[I] = carry[I];
      else fr[I] = fragment<I>(kt, vt);
    });
    __builtin_amdgcn_sched_barrier(0);
    Soft f;
    static_for<SLOTS>([&](auto i) {
      constexpr int I = decltype(i)::value;
      if constexpr (I + PF < SLOTS) {
        fr[I + PF] = fragment<I + PF>(kt, vt);
      } else if constexpr (CARRY_OUT) {
        carry[I + PF - SLOTS] = fragment<I + PF - SLOTS>(kt2, vt2);
      }
      product<I>(fr[I], y, pin);
      soft_slot<I, SLOTS>(f, x, pout);
      __builtin_amdgcn_sched_barrier(0);
    });
    soft_end(f, x, pout);
  }

  // The products of a subtile alone.
  __device__ __forceinline__ void products(floatx16& y, const uint32_t* pin, const char* kt,
                                           const char* vt) {
    u32x4_t fr[SLOTS];
    static_for<PF>([&](auto i) {
      constexpr int I = decltype(i)::value;
      fr[I] = fragment<I>(kt, vt);
    });
    __builtin_amdgcn_sched_barrier(0);
    static_for<SLOTS>([&](auto i) {
      constexpr int I = decltype(i)::value;
      if constexpr (I + PF < SLOTS) fr[I + PF] = fragment<I + PF>(kt, vt);
      product<I>(fr[I], y, pin);
      __builtin_amdgcn_sched_barrier(0);
    });
  }

  // Values of the last subtile.
  __device__ __forceinline__ void last_values(const uint32_t* pin, const char* vt) {
    static_for<SLOTS>([&](auto i) {
      constexpr int I = decltype(i)::value;
      if constexpr (!is_score(I)) {
        floatx16 unused;
        product<I>(fragment<I>(nullptr, vt), unused, pin);
      }
    });
  }
};

// One 64-key tile of the list: its first key, the end of its run, whether some
// key of it is hidden from some row of the workgroup, and whether it renews the
// reference.
struct TileAt {
  int base, end;
  bool masked, renews;
};

// The tiles [first, first + n) of the list that one group of waves walks.
struct GroupTiles {
  const TileList<64>& tl;
  int first, n;
  __device__ __forceinline__ TileAt at(int t, bool renews) const {
    if (t >= n) return {0, 0, false, false};  // nothing to load
    return {tl.base(first + t), tl.end(first + t), tl.masked(first + t), renews};
  }
  // 32-key subtiles; the list's last tile may end within its first half.
  __device__ __forceinline__ int subtiles() const {
    if (n <= 0) return 0;
    return 2 * n - (tl.base(first + n - 1) + 32 >= tl.end(first + n - 1) ? 1 : 0);
  }
};

// Loads of 64-key tiles into the stages of the rolling loop. Wave w of the NW
// that share the stages loads the rows [64 w / NW, 64 (w + 1) / NW) of a tile, one
// 1 KiB block of whole rows per instruction; block i lies i KiB further both in
// memory and in LDS, so the instruction offset serves both and only the lane
// offsets of K, whose chunk permutation has a period of 16 rows, differ from block
// to block.
//
// The waves that share a V stage are NV, at least the NW that share a K stage: the
// two groups of a differential launch read the same values.
template <int D, int NW, int NV>
struct StageLoader {
  using G = TileGeom<D>;
  static constexpr int INSTS = 64 / G::RPI / NW;
  static constexpr int VINSTS = 64 / G::RPI / NV;
  static_assert(VINSTS >= 1, "whole blocks of V per wave");
  static constexpr int KPER = D == 128 ? 4 : 2;  // blocks of the K permutation's period
  static constexpr int NK = INSTS < KPER ? INSTS : KPER;
  __amdgpu_buffer_rsrc_t krs, vrs;
  unsigned koff[NK], voff;
  int row0, vrow0, slot;  // this lane's row in the wave's block 0 of K and V, its 16-byte slot
  int wbase, vwbase;      // byte offset of the wave's first block in a tile (scalar)

  // wave: index among the NW sharing a K stage; vwave: among the NV sharing a V stage.
  __device__ __forceinline__ void init(const uint16_t* kh, const uint16_t* vh, int wave,
                                       int vwave) {
    const int lane = threadIdx.x & 63;
    krs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(kh), (short)0, -1, 0x00020000);
    vrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(vh), (short)0, -1, 0x00020000);
    wbase = wave * INSTS * 1024;
    vwbase = vwave * VINSTS * 1024;
    row0 = wave * INSTS * G::RPI + lane / G::KCH;
    vrow0 = vwave * VINSTS * G::RPI + lane / G::KCH;
    slot = lane % G::KCH;
#pragma unroll
    for (int i = 0; i < NK; ++i)
      koff[i] = row0 * G::ROW + (slot ^ G::swz_k(row0 + i * G::RPI)) * 16;
    voff = vrow0 * G::ROW + (slot ^ G::swz_v(vrow0)) * 16;
  }
  // Block I of a whole tile.
  template <bool ISK, int I>
  __device__ __forceinline__ void block(char* l, unsigned soff) const {
    constexpr int hi = I / 4 * 4096;  // past the 12-bit instruction offset
    if constexpr (ISK)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          krs, (__attribute__((address_space(3))) void*)(l + hi), 16, (int)koff[I % NK],
          (int)(soff + hi), I % 4 * 1024, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          vrs, (__attribute__((address_space(3))) void*)(l + hi), 16, (int)voff,
          (int)(soff + hi), I % 4 * 1024, 0);
  }
  template <bool ISK>
  __device__ __forceinline__ void load(char* stage, int kb, int kend) const {
    const int nrows = kend - kb;
    if (nrows <= 0) return;  // a tile past the last one
    constexpr int N = ISK ? INSTS : VINSTS;
    char* l = stage + (ISK ? wbase : vwbase);
    const unsigned soff = (unsigned)kb * G::ROW;
    if (nrows >= 64) {
      static_for<N>([&](auto q) { block<ISK, decltype(q)::value>(l, soff); });
    } else {
      // Ragged tile: rows past the run repeat its last row (masked later).
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int r = (ISK ? row0 : vrow0) + i * G::RPI;
        const int c = slot ^ (ISK ? G::swz_k(r) : G::swz_v(r));
        const int off = min(r, nrows - 1) * G::ROW + c * 16;
        auto* d = (__attribute__((address_space(3))) void*)(l + i * 1024);
        if constexpr (ISK)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(krs, d, 16, off, (int)soff, 0, 0);
        else
          __builtin_amdgcn_raw_ptr_buffer_load_lds(vrs, d, 16, off, (int)soff, 0, 0);
      }
    }
  }
};

// One step of the rolling loop, tiles t0 = u, t1 = u + 1, t2 = u + 2: the softmax
// of the second half of tile u (scores in xa) and of the first half of tile u + 1
// (xb, if `second`), beside the scores of tile u + 1 (K stage `knext`) and the
// values of tile u (V stage `vcur`, weights of its first half in pb on entry).
// Meanwhile K of tile u + 2 and V of tile u + 1 land in the two stages nobody
// reads during the step. With RENEW a tile u + 1 may renew the reference: then its
// weights wait for both halves of its scores and all values of tile u.
template <int D, int NW, int NV, bool RENEW>
__device__ __forceinline__ void pair_step(char* knext, char* kfree, char* vcur, char* vfree,
                                          Rolling<D>& ro, const StageLoader<D, NW, NV>& ld,
                                          const TileAt& t0, TileAt& t1, const TileAt& t2,
                                          bool second, float& top, int lim, int lo, int sinks,
                                          int h, floatx16& xa, floatx16& xb, uint32_t* pa,
                                          uint32_t* pb) {
  using R = Rolling<D>;
  constexpr int SUB = TileGeom<D>::SUB;
  u32x4_t carry[R::PF];
  ld.template load<true>(kfree, t2.base, t2.end);
  ld.template load<false>(vfree, t1.base, t1.end);
  if (t0.masked) mask_scores(xa, t0.base + 32, t0.end, lim, lo, sinks, h);
  ro.template subtile<false, true>(xa, xb, pb, pa, knext, vcur, knext + SUB, vcur + SUB, carry);
  const bool renews = RENEW && __builtin_expect(t1.renews, 0);
  if (second && !renews) {
    if (t1.masked) mask_scores(xb, t1.base, t1.end, lim, lo, sinks, h);
    ro.template subtile<true, false>(xb, xa, pa, pb, knext + SUB, vcur + SUB, nullptr, nullptr,
                                     carry);
  }
  if (renews) {
    ro.products(xa, pa, knext + SUB, vcur + SUB);
    if (t1.masked) {
      mask_scores(xb, t1.base, t1.end, lim, lo, sinks, h);
      mask_scores(xa, t1.base + 32, t1.end, lim, lo, sinks, h);
      t1.masked = false;  // both halves are
    }
    ro.renew(top, xb, xa, pb);
  }
}

// Forms of the kernel.
enum Form {
  kStream,    // streaming loop (split producer of decode shapes)
  kRolling,   // rolling loop
  kKeySplit,  // rolling loop, two groups of waves over the two halves of the key tiles
  kDiffPair,  // rolling loop, two groups of waves over the two branches of a
              // differential layer
  kDiffRenew,  // kDiffPair whose rows renew their reference every a.renew tiles
};

// NW waves (of 32 query rows each) per group; the two-group forms hold two
// groups over the same rows, with stages of their own, that meet in LDS at the
// end.
//
// kKeySplit serves grids that leave the chip's SIMDs without a second wave: one
// wave alone reaches 88% of the rate of two on a SIMD, so what such a launch
// waits for is the chain of a workgroup's tiles, and two groups halve it. 8 heads
// of 64, 2048 causal: 28.3 -> 17.7 us; 32/8 heads of 128, 4 x 100 of 1500 keys:
// 30.2 -> 22.5 us (the rule that selects it holds both sides' figures).
//
// kDiffPair runs both branches of a differential layer in one launch: the
// second branch's output stays in registers and LDS instead of going through o
// between two launches, and each V tile is staged once for both. 32/8 heads of
// 128, 1024 causal: 52.5 -> 37.0 us, 4 x 1024: 118.5 -> 105.8 us; 32 heads, 1024 of
// 32768 keys: 1003 us in two split branches, 999 in one launch, 968 with the
// shared V stages. Grids of thousands of row tiles of grouped heads of 64 lose up
// to 3% against a launch per branch, whose four-wave workgroups run three waves to
// a SIMD: 15 x 32/8 heads, 1321 of 2227 keys 715 us before, 734 now, 11 x 64/8, 762
// of 886 245 and 252 (ungrouped heads gain there too: 4 x 32, 1024 87 and 82).
//
// kDiffRenew is kDiffPair where the launch takes the place of a split call: every
// a.renew key tiles, the tiles of one of the split's partitions, a row's reference
// starts again at the maximum of a 64-key tile, as each partition's would, so the
// weights are rounded to bf16 as the split rounds them. The renewal stands behind
// the step in a block of its own: as an else of the step's second half it cost 87
// spilled registers, inside the second half 4% on every step. It costs a step of
// its own, 1-1.5 us: 32 heads, 1024 of 32768 keys, every 256 tiles 986 us without,
// 992 with it; 32/8 heads of 64, 768 of 3000 keys, every 32 tiles 55.7, 57.9; 12
// heads of 64, 128 of 640 keys, every tile 17.6, 22.2.
//
// Occupancy target: two waves per SIMD (two workgroups of four waves per CU, four
// of the streaming loop's two-wave ones, overlap each other's barrier and
// latency stalls; a workgroup of eight waves has both on its own), three at D = 64
// where the registers allow; the four-wave two-group form and the two-wave
// workgroup of the rolling loop serve grids too small for that.
template <int D, int NW, Form F>
__global__ __launch_bounds__(NW * 64 * (F >= kKeySplit ? 2 : 1))
__attribute__((amdgpu_waves_per_eu(NW == 2 && F != kStream         ? 1
                                   : D == 64 && F < kKeySplit ? 3
                                                              : 2)))
void attn_mfma_kernel(MfmaParams a) {
  using Geo = TileGeom<D>;
  constexpr bool STREAM = F == kStream;
  constexpr bool DIFF = F >= kDiffPair, RENEW = F == kDiffRenew;
  constexpr int GROUPS = F >= kKeySplit ? 2 : 1;
  constexpr int KSTEPS = D / 16;
  constexpr int DT = D / 32;
  constexpr int BM = 32 * NW;
  constexpr int BN = STREAM ? 32 : 64;  // keys per tile

  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = GROUPS > 1 ? wid / NW : 0;  // group of this wave
  const int wave = wid - grp * NW;            // wave inside the group
  const int h = lane >> 5;   // k-group of the MFMA operands
  const int ql = lane & 31;  // this lane's query inside the wave's 32 rows

  // Workgroup -> (row tile, partition, b*Hkv). Workgroups are dispatched to the
  // chip's 8 XCDs round-robin by linear id; the id is remapped so that each XCD
  // receives a contiguous run of kv heads, and all row tiles of a head, which
  // read the same K/V, share one XCD's L2. Row tiles are visited last-first so
  // causal tiles with the most keys start first: head by head, or (a.interleave)
  // over all heads of the XCD, which leaves only short tiles for the end.
  const unsigned nwg = gridDim.x * gridDim.y * gridDim.z;
  unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  if (nwg % kXcds == 0) lin = (lin % kXcds) * (nwg / kXcds) + lin / kXcds;
  int mt = a.mtiles - 1 - (int)(lin % gridDim.x);
  const int p = (int)((lin / gridDim.x) % gridDim.y);
  int bh = (int)(lin / (gridDim.x * gridDim.y));
  if (a.interleave) {
    const unsigned heads = gridDim.z / kXcds, wgs = nwg / kXcds;  // of one XCD
    mt = a.mtiles - 1 - (int)(lin % wgs / heads);
    bh = (int)(lin / wgs * heads + lin % wgs % heads);
  }
  const int b = bh / a.Hkv, hkv = bh % a.Hkv;

  const size_t kvhead = ((size_t)b * a.Hkv + hkv) * (size_t)a.Skv * D;
  const uint16_t* kh = (DIFF && grp ? a.k2 : a.k) + kvhead;
  const uint16_t* vh = a.v + kvhead;

  // This lane's query row.
  const int r = mt * BM + wave * 32 + ql;
  const bool rvalid = r < a.R;
  const int sq = rvalid ? r / a.G : 0;
  const int g = rvalid ? r % a.G : 0;
  const size_t orow = (((size_t)b * a.Hq + (size_t)hkv * a.G + g) * a.Sq + sq);
  const int off = a.Skv - a.Sq;
  const int lim = !rvalid ? -1 : (a.causal ? sq + off : 0x7fffffff);
  const int W = a.runs.window;
  const int lo = W > 0 ? lim - W : INT_MIN;  // keys at or left of lo are outside the window

  // Key tiles of this workgroup. The partition is a range [v0, v1) of the
  // virtual key axis (the sink run [0, la) followed by the window run from key
  // bs); its part in each run is cut at the last key any row can see and, in
  // the window run, at the first key of the earliest row's window.
  TileList<BN> tl;
  {
    const int la = a.runs.la, bs = a.runs.bs;
    const int v0 = p * a.T;
    const int v1 = min(v0 + a.T, a.runs.lv);
    int cend = 0x7fffffff, wbeg = 0;
    tl.full_lo = 0x7fffffff;
    tl.win_lo = INT_MIN;
    if (a.causal) {
      const int r_lo = mt * BM;
      const int r_hi = min(mt * BM + BM, a.R) - 1;
      tl.full_lo = r_lo / a.G + off;
      cend = r_hi / a.G + off + 1;
      if (W > 0) {
        wbeg = max(0, tl.full_lo - W + 1) / BN * BN;
        tl.win_lo = r_hi / a.G + off - W + 1;
      }
    }
    tl.a0 = v0;
    tl.aend = min(min(v1, la), cend);
    tl.na = tl.aend > tl.a0 ? (tl.aend - tl.a0 + BN - 1) / BN : 0;
    tl.b0 = max(bs + max(v0, la) - la, wbeg);
    tl.bend = min(bs + v1 - la, cend);
    tl.n = tl.na + (tl.bend > tl.b0 ? (tl.bend - tl.b0 + BN - 1) / BN : 0);
    tl.sinks = W > 0 ? a.runs.sinks : 0;
  }
  const int ntiles = tl.n;

  // Q^T fragments (B operand): lane holds q[row][16*s + 8*h .. +8].
  bf16x8_t qf[KSTEPS];
  {
    const u32x4_t* qp =
        reinterpret_cast<const u32x4_t*>((DIFF && grp ? a.q2 : a.q) + orow * D);
    const u32x4_t zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) {
      const u32x4_t x = (rvalid ? qp[2 * s + h] : zero) ^ a.qflip;
      qf[s] = __builtin_bit_cast(bf16x8_t, x);
    }
  }

  floatx16 oacc[DT];
#pragma unroll
  for (int i = 0; i < DT; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) oacc[i][j] = 0.f;
  float mref = STREAM ? kNegInf : kNoRef;  // reference maximum, base-2 units
  float lsum = 0.f;      // this lane's half of the row sum
  // The floor keeps a zero scale well defined: every visible key gets weight 1
  // (2^(x c) rounds to 1 for any finite score), while a hidden key's -inf stays
  // -inf instead of becoming -inf * 0 = NaN.
  const float c = fmaxf(a.c_abs, 1e-30f);
  // Per-lane LDS byte offsets of the fragment reads inside a stage: K row ql,
  // chunk 2s + h of k-step s; and, per 32-column tile dt of V^T, the
  // transposing-read pointer of this lane (row 4(lane/32) + (lane%16)/4 of a
  // 16-key step, 8 bytes at column 32 dt + 16 ((lane/16)%2) + 4 (lane%4)).
  int kread[KSTEPS];
#pragma unroll
  for (int s = 0; s < KSTEPS; ++s) kread[s] = ql * Geo::ROW + ((2 * s + h) ^ Geo::swz_k(ql)) * 16;
  int vread[DT];
  {
    const int j16 = lane & 15, grp = lane >> 4;
    const int vr = 4 * (grp >> 1) + (j16 >> 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const int d_off = 32 * dt + 16 * (grp & 1) + 4 * (j16 & 3);
      vread[dt] = vr * Geo::ROW + (((d_off >> 3) ^ Geo::swz_v(vr)) * 16) + 2 * (d_off & 7);
    }
  }

  if constexpr (STREAM) {
    // Prologue: K and V of tile 0 into stage 0, K of tile 1 into K stage 1, then
    // tile 0's scores; the second barrier orders those K reads before stage 0 is
    // rewritten by the first step.
    __shared__ __align__(1024) char smem[4 * Geo::SUB];
    Loader<D, NW> ld;
    ld.init();
    floatx16 sacc[2];  // S^T of the current and the next tile
    if (ntiles > 0) {
      ld.template load_k<0>(smem, kh, tl.base(0), tl.end(0));
      ld.template load_v<0>(smem, vh, tl.base(0), tl.end(0));
      ld.template load_k<1>(smem, kh, tl.base(1), tl.end(1));
    }
    wait_tile_loads();
    __syncthreads();
    if (ntiles > 0) subtile_scores<D>(smem + Geo::template k_off<0>(), kread, qf, sacc[0]);
    __syncthreads();
    for (int j = 0; j < ntiles; j += 2) {
      pipelined_step<D, NW, 0>(smem, ld, kh, vh, tl, j, lim, lo, h, kread, vread, qf, sacc, oacc,
                               lsum, mref, c);
      if (j + 1 < ntiles)
        pipelined_step<D, NW, 1>(smem, ld, kh, vh, tl, j + 1, lim, lo, h, kread, vread, qf, sacc,
                                 oacc, lsum, mref, c);
    }
  }

  // Output rows: value / sum, or the state of the partition, of the value tiles
  // [DT0, DT0 + NDT) (32 channels each; lane halves hold alternate 4-channel runs).
  auto store = [&](const floatx16* val, int dt0, auto ndt, float ref, float ltot) {
    constexpr int NDT = decltype(ndt)::value;
    if (!rvalid) return;
    auto put = [&](float* dst, float mul) {
#pragma unroll
      for (int i = 0; i < NDT; ++i)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          *reinterpret_cast<float4*>(dst + (dt0 + i) * 32 + 8 * q4 + 4 * h) =
              make_float4(val[i][4 * q4] * mul, val[i][4 * q4 + 1] * mul, val[i][4 * q4 + 2] * mul,
                          val[i][4 * q4 + 3] * mul);
    };
    if (a.ws_m == nullptr) {
      put(a.o + orow * D, ltot > 0.f ? 1.f / ltot : 0.f);
    } else {
      const size_t slot = orow * (size_t)a.P + p;
      if (h == 0) {
        // Reference in natural-log units, in terms of scale * q.k.
        a.ws_m[slot] = ref == kNegInf || ref == kNoRef ? kNegInf : ref * kLn2;
        a.ws_l[slot] = ltot;
      }
      put(a.ws_acc + slot * D, 1.f);
    }
  };

  if constexpr (STREAM) {
    store(oacc, 0, std::integral_constant<int, DT>{}, mref, lsum + __shfl_xor(lsum, 32, 64));
    return;
  } else {
    // The four stages are objects of their own, and the loads go through buffer
    // descriptors: the compiler then neither waits for a step's loads before its
    // first reads (they cannot alias) nor drains the LDS counter at every read
    // (it does with a flat direct-to-LDS load in flight).
    constexpr int STAGE = 2 * Geo::SUB;  // one group's bytes of a stage
    // The two branches of a differential launch share the V stages.
    constexpr int VGROUPS = DIFF ? 1 : GROUPS, NV = NW * GROUPS / VGROUPS;
    __shared__ __align__(1024) char sk0[GROUPS * STAGE], sk1[GROUPS * STAGE];
    __shared__ __align__(1024) char sv0[VGROUPS * STAGE], sv1[VGROUPS * STAGE];
    char* const k0 = sk0 + grp * STAGE;
    char* const k1 = sk1 + grp * STAGE;
    char* const v0 = sv0 + (VGROUPS > 1 ? grp * STAGE : 0);
    char* const v1 = sv1 + (VGROUPS > 1 ? grp * STAGE : 0);
    // Tiles of this group, and the steps the workgroup's barriers count: those of
    // the first half of the tiles, which is never the shorter one.
    const int first_half = (ntiles + 1) / 2;
    const GroupTiles gt{tl, F == kKeySplit && grp ? first_half : 0,
                        F != kKeySplit ? ntiles : grp ? ntiles - first_half : first_half};
    const int nsub = gt.subtiles();
    const int steps =
        F == kKeySplit ? GroupTiles{tl, 0, first_half}.subtiles() / 2 : nsub / 2;
    floatx16 xa, xb;        // scores of odd and even subtiles
    uint32_t pa[8], pb[8];  // their weights
    Rolling<D> ro{kread, vread, qf, oacc, lsum, mref, c};
    if (ntiles > 0) {
      StageLoader<D, NW, NV> ld;
      ld.init(kh, vh, wave, DIFF ? wid : wave);
      int due = RENEW ? a.renew : 0;  // tiles until the next one that renews
      float top = kNoRef;
      auto tile = [&](int t) {  // t = 1, 2, 3, ...
        const bool renews = RENEW && --due == 0;
        if (renews) due = a.renew;
        return gt.at(t, renews);
      };
      TileAt t0 = gt.at(0, false), t1 = tile(1), t2;
      // Prologue: tile 0's K and V and tile 1's K; tile 0's scores, then subtile 0's
      // softmax. The second barrier orders those K reads before stage 0 is rewritten
      // by the first step.
      ld.template load<true>(k0, t0.base, t0.end);
      ld.template load<false>(v0, t0.base, t0.end);
      ld.template load<true>(k1, t1.base, t1.end);
      wait_tile_loads();
      __syncthreads();
      if (GROUPS == 1 || nsub > 0) {
        tile_scores<D>(k0, kread, qf, xb, xa);
        if (t0.masked) {
          mask_scores(xb, t0.base, t0.end, lim, lo, tl.sinks, h);
          mask_scores(xa, t0.base + 32, t0.end, lim, lo, tl.sinks, h);
          t0.masked = false;  // both halves are
        }
        ro.start(xb, xa, pb);
      }
      __syncthreads();
      for (int u = 0; u < steps; u += 2) {
        t2 = tile(u + 2);
        if (GROUPS == 1 || 2 * u + 1 < nsub)
          pair_step<D, NW, NV, RENEW>(k1, k0, v0, v1, ro, ld, t0, t1, t2, 2 * u + 2 < nsub, top,
                                      lim, lo, tl.sinks, h, xa, xb, pa, pb);
        wait_tile_loads();
        __syncthreads();
        if (u + 1 >= steps) break;
        t0 = tile(u + 3);
        if (GROUPS == 1 || 2 * u + 3 < nsub)
          pair_step<D, NW, NV, RENEW>(k0, k1, v1, v0, ro, ld, t1, t2, t0, 2 * u + 4 < nsub, top,
                                      lim, lo, tl.sinks, h, xa, xb, pa, pb);
        wait_tile_loads();
        __syncthreads();
        t1 = t0;
        t0 = t2;
      }
      if (GROUPS == 1 || nsub > 0) {
        const int last = nsub - 1;
        const char* vl = (last >> 1 & 1) ? v1 : v0;
        if (last & 1)
          ro.last_values(pa, vl + Geo::SUB);
        else
          ro.last_values(pb, vl);
      }
    }
    const float ltot = lsum + __shfl_xor(lsum, 32, 64);  // both lane halves of the row
    if constexpr (GROUPS == 1) {
      store(oacc, 0, std::integral_constant<int, DT>{}, mref, ltot);
    } else {
      // The groups meet: each sends the other half of its value tiles (and its
      // reference and sum), and finishes its own half of the channels.
      constexpr int HT = DT / 2;
      const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
      float4* out = reinterpret_cast<float4*>(grp ? sk1 : sk0) + wave * (HT * 4 * 64) + lane;
      const float4* in =
          reinterpret_cast<const float4*>(grp ? sk0 : sk1) + wave * (HT * 4 * 64) + lane;
      float2* ml = reinterpret_cast<float2*>(sv0);  // [group][wave][lane]
      float* sq2 = reinterpret_cast<float*>(sv1);   // [group][wave][lane]
      floatx16 own[HT];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < HT; ++i) {
#pragma unroll
        for (int e = 0; e < 16; ++e) own[i][e] = grp ? oacc[HT + i][e] : oacc[i][e];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          float x[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x[e] = grp ? oacc[i][4 * q4 + e] : oacc[HT + i][4 * q4 + e];
            if constexpr (DIFF) x[e] *= inv;
          }
          out[(i * 4 + q4) * 64] = make_float4(x[0], x[1], x[2], x[3]);
        }
      }
      ml[(grp * NW + wave) * 64 + lane] = make_float2(mref, ltot);
      __syncthreads();
      if constexpr (F == kKeySplit) {
        const float2 other = ml[((1 - grp) * NW + wave) * 64 + lane];
        const float ref = fmaxf(mref, other.x);
        const float wo = exp2_fast(mref - ref), wi = exp2_fast(other.x - ref);
        const float lt = fmaf(other.y, wi, ltot * wo);
#pragma unroll
        for (int i = 0; i < HT; ++i)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const float4 x = in[(i * 4 + q4) * 64];
            own[i][4 * q4] = fmaf(x.x, wi, own[i][4 * q4] * wo);
            own[i][4 * q4 + 1] = fmaf(x.y, wi, own[i][4 * q4 + 1] * wo);
            own[i][4 * q4 + 2] = fmaf(x.z, wi, own[i][4 * q4 + 2] * wo);
            own[i][4 * q4 + 3] = fmaf(x.w, wi, own[i][4 * q4 + 3] * wo);
          }
        store(own, grp * HT, std::integral_constant<int, HT>{}, ref, lt);
      } else {
        // y = A1 - lambda A2 (the first group holds the first branch), then the
        // RMS normalisation of the row over all channels.
        const float lam = diff_lambda(a.diff, lane, D);
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < HT; ++i)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const float4 x4 = in[(i * 4 + q4) * 64];
            const float x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float mine = own[i][4 * q4 + e] * inv;
              const float y = fmaf(-lam, grp ? mine : x[e], grp ? x[e] : mine);
              own[i][4 * q4 + e] = y;
              ss = fmaf(y, y, ss);
            }
          }
        ss += __shfl_xor(ss, 32, 64);
        sq2[(grp * NW + wave) * 64 + lane] = ss;
        __syncthreads();
        ss += sq2[((1 - grp) * NW + wave) * 64 + lane];
        const float rn = diff_row_factor(a.diff, ss, D);
        if (!rvalid) return;
        float* orp = a.o + orow * D;
#pragma unroll
        for (int i = 0; i < HT; ++i)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const int d = (grp * HT + i) * 32 + 8 * q4 + 4 * h;
            const float4 gw = *reinterpret_cast<const float4*>(a.diff.gamma + d);
            *reinterpret_cast<float4*>(orp + d) =
                make_float4(rn * gw.x * own[i][4 * q4], rn * gw.y * own[i][4 * q4 + 1],
                            rn * gw.z * own[i][4 * q4 + 2], rn * gw.w * own[i][4 * q4 + 3]);
          }
      }
    }
  }
}

template <int D, int NW, Form F>
hipError_t launch_one(const MfmaParams& a, hipStream_t stream) {
  hipLaunchKernelGGL((attn_mfma_kernel<D, NW, F>), dim3(a.mtiles, a.P, a.B * a.Hkv),
                     dim3(NW * 64 * (F >= kKeySplit ? 2 : 1)), 0, stream, a);
  return hipGetLastError();
}

template <int D>
hipError_t launch_d(const MfmaParams& a, hipStream_t stream) {
  if (a.diff.gamma != nullptr) {
    if (a.renew > 0)
      return a.bm == 64 ? launch_one<D, 2, kDiffRenew>(a, stream)
                        : launch_one<D, 4, kDiffRenew>(a, stream);
    return a.bm == 64 ? launch_one<D, 2, kDiffPair>(a, stream)
                      : launch_one<D, 4, kDiffPair>(a, stream);
  }
  if (a.key_split) return launch_one<D, 2, kKeySplit>(a, stream);
  if (a.bm == 128) return launch_one<D, 4, kRolling>(a, stream);
  // The split producer with one 64-row tile per kv head (decode shapes) streams:
  // its loads assume that every key is read once.
  if (a.mtiles == 1 && a.ws_m != nullptr) return launch_one<D, 2, kStream>(a, stream);
  return launch_one<D, 2, kRolling>(a, stream);
}

}  // namespace

hipError_t launch_mfma_attention(const MfmaParams& a, hipStream_t stream) {
  if (a.bm != 64 && a.bm != 128) return hipErrorInvalidValue;
  return a.D == 128 ? launch_d<128>(a, stream) : launch_d<64>(a, stream);
}

}  // namespace ef
