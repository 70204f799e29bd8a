// HIP kernels of the layer-wise Top-K compressor on gfx950 (CDNA4, wave64).
//
// C(v) keeps the k_l elements of largest |v| of each tensor (equal
// magnitudes: the lower index first) and zeroes the others.  The kept set of
// each (row, tensor) is found on the 31-bit key |v| (the bit pattern of a
// non-negative float orders like its value):
//   histogram  the pass that forms Delta (one workgroup per tile and row)
//              also counts the keys into a tile histogram (LDS atomics,
//              16-bit counts stored), fine around the (row, tensor)'s
//              previous threshold and coarser away from it, and writes the
//              tile's speculative list (the elements at or above a bound just
//              below the previous threshold);
//   sum        tile histograms of large tensors are added per group of 64
//              tiles (and groups per super-group for very large tensors);
//   pick       a workgroup per (row, tensor) finds the bin b1 that holds the
//              k-th largest key.  A small tensor (up to 64 tiles; up to 16 in
//              a plan that has larger ones) it selects as a whole, so its
//              selection is this one kernel;
//   refine     (plans with a tensor of more than 4096 tiles) a bin b1 with
//              many elements is narrowed to a sub-range of it, 11 key bits at
//              a time, by the workgroups of all tiles;
//   gather     the elements of b1 (the candidates) of large tensors, tile by
//              tile, and each tile's count of elements above b1: from the
//              tile's list when its bound lies at or below b1, else from one
//              more read of Delta (a full b1 is narrowed by 11 key bits first);
//   select     a workgroup per (row, large tensor) finds, among the
//              candidates only, the threshold key tau and the last kept index
//              iota of the elements equal to tau, and turns the tiles' counts
//              into each tile's first rank;
//   emit       one wave per tile writes its selection words, rank words and
//              kept values in index order, and sets the kept elements of the
//              error to 0 (e = Delta - C(Delta) is Delta elsewhere), from the
//              tile's list when it reaches down to tau, else from one more
//              read of Delta.
// All of it is integer counting, so the kept set does not depend on the
// launch geometry, nor on the order in which candidates are collected.
//
// The streaming passes (Delta, gather) run one short-lived workgroup or wave
// per 2048-element tile: on MI355X a 2-read/1-write stream reaches about
// 6.1 TB/s that way and about 5.1 TB/s when each workgroup walks 64Ki
// elements.
//
// The server runs the same steps on its one row (row k_max of the scratch)
// after k_tk_aggregate has formed Delta = e_srv + mean of the K messages.
#include "saef_device.h"
#include "saef_topk.h"

namespace saef {
namespace {

constexpr uint32_t kFiniteLimit = 0x7F800000u;  // keys >= this are Inf or NaN
constexpr int kTkU = 8;                         // words per wave per pass (Delta pass: one pass)
constexpr int kTileWords = kTkTileElems / 64;     // 32
// Threads of the server aggregation: a wave per tile of a chunk.
constexpr int kAgg = kTkChunk / kTkTileElems * kWave;
static_assert(kTileWords <= kWave, "one selection word of a tile per lane");
// Word 3 of a raw buffer descriptor on gfx9 parts (32-bit data format, no
// swizzle, no index stride).  A load through a raw buffer resource of n
// bytes returns 0 for a byte offset at or past n, without touching memory.
constexpr int kBufWord3 = 0x00020000;

__device__ __forceinline__ uint32_t key_of(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }

// The mid bins of a side, in far bins.
constexpr int kMidFarB = kTkMidB >> (kTkFarShift - kTkMidShift);
constexpr int kMidFarA = kTkMidA >> (kTkFarShift - kTkMidShift);

// Pass-1 bin of a key for the near range [win, win + kTkNear bins).  Bins
// order like the keys.
__device__ __forceinline__ uint32_t hist_bin(uint32_t key, uint32_t win) {
  const int32_t s = (int32_t)(key - win);  // keys and win are below 2^31
  // below: x keys between key and win; above: x keys past the near range
  const uint32_t xb = ~(uint32_t)s, xa = (uint32_t)s - ((uint32_t)kTkNear << kTkSubShift);
  const uint32_t mb = xb >> kTkMidShift, ma = xa >> kTkMidShift;
  const uint32_t gb = mb < (uint32_t)kTkMidB
                          ? mb : min((xb >> kTkFarShift) + (uint32_t)(kTkMidB - kMidFarB),
                                     (uint32_t)(kTkBelow - 1));
  const uint32_t ga = ma < (uint32_t)kTkMidA
                          ? ma : min((xa >> kTkFarShift) + (uint32_t)(kTkMidA - kMidFarA),
                                     (uint32_t)(kTkAbove - 1));
  const uint32_t side = s < 0 ? (uint32_t)(kTkBelow - 1) - gb : (uint32_t)(kTkBelow + kTkNear) + ga;
  const uint32_t d = (uint32_t)s >> kTkSubShift;
  return d < (uint32_t)kTkNear ? (uint32_t)kTkBelow + d : side;
}

// The near range of the next call: from kTkSpecMargin under tau on.
__device__ __forceinline__ uint32_t window_for(uint32_t tau) {
  return tau > kTkSpecMargin ? tau - kTkSpecMargin : 0u;
}

__device__ __forceinline__ uint16_t* tile_hist(const TkDev& tk, const DevLayout& lay, int row,
                                               int64_t ti) {
  return tk.thist + ((int64_t)row * lay.n_tiles + ti) * kTkHistPad;
}

// Stores an LDS histogram of kTkHistPad bins as 16-bit counts, two per store.
__device__ __forceinline__ void store_hist16(const uint32_t* h, uint16_t* out) {
  for (int i = threadIdx.x; i < kTkHistPad / 2; i += blockDim.x)
    reinterpret_cast<uint32_t*>(out)[i] = (h[2 * i] & 0xFFFFu) | (h[2 * i + 1] << 16);
}

// Lower key bound of the speculative lists of a (row, tensor): the previous
// threshold key minus the margin; 2^31 (no element) before the first
// threshold or when the tensor keeps no lists.
__device__ __forceinline__ uint32_t spec_floor(const TkSel& st) {
  if (st.tau == 0u || st.lists == 0u) return 0x80000000u;
  return st.tau > kTkSpecMargin ? st.tau - kTkSpecMargin : 0u;
}

// ------------------------------------------------------------------ pass 1 (workers)
// A wave's loads of one worker's tile (kTkU words from w0 on; buffer
// resources over the tile, so lanes past its end load 0), issued before the
// histogram is cleared and waited for after it.
template <bool kMom, bool kPend, bool kXh>
struct DeltaLoads {
  float g[kTkU], e[kTkU], m[kTkU], x[kTkU];
  u64 pend[kTkU];

  __device__ __forceinline__ DeltaLoads(int w0, int nw, Buf rg, Buf re, Buf rm, Buf rx,
                                        const uint64_t* __restrict__ pk) {
    const uint32_t off0 = (uint32_t)(w0 * 64 + lane_id()) * 4u;
#pragma unroll
    for (int u = 0; u < kTkU; ++u) {
      g[u] = buf_ld(rg, off0 + 256u * u);
      e[u] = buf_ld(re, off0 + 256u * u);
      m[u] = kMom ? buf_ld(rm, off0 + 256u * u) : 0.0f;
      x[u] = kXh ? buf_ld_cached(rx, off0 + 256u * u) : 0.0f;
      pend[u] = kPend ? ld_word_ro(pk + min(w0 + u, nw - 1)) : 0ull;
    }
  }
};

// kTkU words of one worker's tile: m <- fma(mu, m, g) with kMom, Delta =
// fma(lr, m or g, e), Delta stored into e, its key counted; kXh: xh = x - e
// from the same read of e.
template <bool kMom, bool kPend, bool kXh, bool kFull>
__device__ __forceinline__ void delta_words(const DeltaLoads<kMom, kPend, kXh>& ld, int w0,
                                            int count, float lr, float mu, Buf rm, Buf re, Buf rh,
                                            uint32_t win, uint32_t lo, uint32_t* h,
                                            uint32_t (&bits)[kTkU], u64 (&lm)[kTkU], bool& bad) {
  const int lane = lane_id();
  const uint32_t off0 = (uint32_t)(w0 * 64 + lane) * 4u;
  // keys in the open low bin, counted without LDS atomics: most of them when the
  // values fall (resnet50 K = 8 Top-1%, all divided by 16: 1340 us a call before,
  // 1070 now)
  uint32_t low = 0;
#pragma unroll
  for (int u = 0; u < kTkU; ++u) {
    const uint32_t off = off0 + 256u * u;
    const bool ok = kFull || (w0 + u) * 64 + lane < count;
    float ev = ld.e[u];
    if (kPend) ev = sel_by_bit(ld.pend[u], 0.0f, ev);  // kept by the previous call: 0
    if (kXh) buf_st(rh, off, ld.x[u] - ev);            // x^(k)_{t+1/2} = x_t - e^(k)_t
    float step = ld.g[u];
    if (kMom) {
      step = __builtin_fmaf(mu, ld.m[u], ld.g[u]);  // m^(k)_{t+1} = mu m^(k)_t + grad
      buf_st(rm, off, step);
    }
    const float p = __builtin_fmaf(lr, step, ev);  // Delta^(k) = e^(k) + lr m^(k)_{t+1}
    const uint32_t key = key_of(p);
    bits[u] = __float_as_uint(p);
    lm[u] = __ballot(ok && key >= lo);
    buf_st(re, off, p);
    const uint32_t bin = hist_bin(key, win);
    low += (uint32_t)__popcll(__ballot(ok && bin == 0u));
    if (!ok) continue;
    bad |= key >= kFiniteLimit;
    if (bin != 0u) atomicAdd(&h[bin], 1u);
  }
  if (low != 0u && lane == 0) atomicAdd(&h[0], low);
}

// Grid: run_padded_tiles(p.t1 - p.t0) * R workgroups; workgroup b handles one
// (tile, row) in the XCD-aware order of run_tile_of over the part's tiles (the
// rows of a run of tiles follow one another on one XCD and share x there).
// Each wave takes kTkU words of the tile (one pass); the tile's speculative
// list is written in index order (wave by wave) when it fits.  kPend: e
// holds the previous call's Delta with its kept elements (selection words
// psel) still to be set to 0; they are read as 0.  kXh: also the iteration's
// step ahead xh = x - e (the gradient is in place before it): 16 bytes per
// element for 20 in two kernels.
template <bool kMom, bool kPend, bool kXh>
__global__ __launch_bounds__(kBlock) void k_tk_delta(DevLayout lay, TkDev tk, TkPart p, int R,
                                                     int row0,
                                                     float lr, float mu,
                                                     const float* __restrict__ g,
                                                     float* __restrict__ m,
                                                     float* __restrict__ e,
                                                     const uint64_t* __restrict__ psel,
                                                     const float* __restrict__ x,
                                                     float* __restrict__ xh) {
  static_assert(kWaves * kTkU == kTileWords, "one pass of the four waves covers a tile");
  __shared__ uint32_t h[kTkHistPad];
  __shared__ uint32_t s_cnt[kWaves];
  int r;
  int64_t tl;
  run_tile_of(blockIdx.x, R, tile_run_shift(p.t1 - p.t0), r, tl);
  if (tl >= p.t1 - p.t0) return;
  const int k = row0 + r;
  const int64_t ti = p.t0 + tl;
  const Tile tile = lay.tiles[ti];
  const TkSel* st = tk.sel + (int64_t)k * lay.L + tile.l;
  const int64_t row = (int64_t)k * lay.d_pad + tile.start;
  const uint32_t nbytes = (uint32_t)tile.count * 4u;
  const Buf rg = buf_of(g + row, nbytes);
  const Buf re = buf_of(e + row, nbytes);
  const Buf rm = buf_of(kMom ? m + row : e + row, nbytes);
  const Buf rx = buf_of(kXh ? x + tile.start : e + row, nbytes);
  const Buf rh = buf_of(kXh ? xh + row : e + row, nbytes);
  const int nw = (tile.count + 63) >> 6;
  const int wave = wave_id();
  const int w0 = wave * kTkU;
  const uint64_t* pk = kPend ? psel + (int64_t)k * (lay.d_pad >> 6) + (tile.start >> 6) : nullptr;
  const DeltaLoads<kMom, kPend, kXh> ld(w0, nw, rg, re, rm, rx, pk);
  const uint32_t win = st->win;
  const uint32_t lo = spec_floor(*st);
  for (int i = threadIdx.x; i < kTkHistPad; i += kBlock) h[i] = 0;
  lds_barrier();
  bool bad = false;
  uint32_t bits[kTkU];  // Delta's bit patterns
  u64 lm[kTkU];
#pragma unroll
  for (int u = 0; u < kTkU; ++u) lm[u] = 0ull;
  if (w0 < nw) {
    if ((w0 + kTkU) * 64 <= tile.count)
      delta_words<kMom, kPend, kXh, true>(ld, w0, tile.count, lr, mu, rm, re, rh, win, lo, h, bits,
                                          lm, bad);
    else
      delta_words<kMom, kPend, kXh, false>(ld, w0, tile.count, lr, mu, rm, re, rh, win, lo, h,
                                           bits, lm, bad);
  }
  if (__ballot(bad) != 0 && lane_id() == 0) atomicOr(lay.status, kStatusRange);
  uint32_t mine = 0;
#pragma unroll
  for (int u = 0; u < kTkU; ++u) mine += (uint32_t)__popcll(lm[u]);
  if (lane_id() == 0) s_cnt[wave] = mine;
  lds_barrier();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    before += w < wave ? s_cnt[w] : 0u;
    total += s_cnt[w];
  }
  // no list (kTkSpecNone) before the first threshold, for a tensor without
  // lists, or when the tile has more than kTkSpecCap such elements
  const bool fits = lo != 0x80000000u && total <= (uint32_t)kTkSpecCap;
  store_hist16(h, tile_hist(tk, lay, k, ti));
  if (threadIdx.x == 0) tk.lcnt[(int64_t)k * lay.n_tiles + ti] = fits ? total : kTkSpecNone;
  if (fits && mine != 0u) {
    u64* out = tk.spec + ((int64_t)k * lay.n_tiles + ti) * kTkSpecCap;
    const int lane = lane_id();
#pragma unroll
    for (int u = 0; u < kTkU; ++u) {
      const uint32_t pos =
          before + __builtin_amdgcn_mbcnt_hi((uint32_t)(lm[u] >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)lm[u], 0u));
      if ((lm[u] >> lane) & 1ull)  // pos < total <= kTkSpecCap
        out[pos] = (u64)bits[u] | ((u64)((w0 + u) * 64 + lane) << 32);
      before += (uint32_t)__popcll(lm[u]);
    }
  }
}

// The sum of the histograms of n <= kN tiles from `first` on (n <= 0: zeros)
// as packed pairs of 16-bit counts: lane holds words lane and lane + 64 of the
// kTkHistPad / 2 of a histogram, every load issued at once.
template <int kN>
__device__ __forceinline__ void tile_hist_sum(const TkDev& tk, const DevLayout& lay, int row,
                                              int64_t first, int n, int lane,
                                              uint32_t (&v)[2]) {
  constexpr int kW = kTkHistPad / 2;
  static_assert(kW == 2 * kWave, "two words per lane");
  const uint32_t* src = reinterpret_cast<const uint32_t*>(tile_hist(tk, lay, row, n > 0 ? first : 0));
  uint32_t a[kN][2];
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    const uint32_t* t = src + (i < n ? i : 0) * kW;
    a[i][0] = t[lane];
    a[i][1] = t[lane + kWave];
  }
  v[0] = v[1] = 0;
#pragma unroll
  for (int i = 0; i < kN; ++i)
#pragma unroll
    for (int q = 0; q < 2; ++q) v[q] += i < n ? a[i][q] : 0u;
}
// Adds a wave's packed sums to the histogram h in LDS.
__device__ __forceinline__ void tile_hist_add(uint32_t* h, int lane, const uint32_t (&v)[2]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int w = lane + q * kWave;
    if ((v[q] & 0xFFFFu) != 0u) atomicAdd(&h[2 * w], v[q] & 0xFFFFu);
    if ((v[q] >> 16) != 0u) atomicAdd(&h[2 * w + 1], v[q] >> 16);
  }
}

// ------------------------------------------------------------------ sums
// Grid: R * n workgroups, n the part's groups (kSuper: super-groups).
// Workgroup b adds the tile histograms of the part's group b % n (or the
// group sums of its super-group b % n) of row row0 + b / n.  Tile histograms:
// each wave takes 16 tiles with all its loads in flight at once and adds them
// as pairs of 16-bit counts (16 tiles of 2048 elements do not overflow one).
template <bool kSuper>
__global__ __launch_bounds__(kBlock) void k_tk_sum(DevLayout lay, TkDev tk, TkPart p, int row0) {
  const int64_t n = kSuper ? p.s1 - p.s0 : p.g1 - p.g0;
  const int64_t gi = (kSuper ? p.s0 : p.g0) + (int64_t)(blockIdx.x % n);
  const int row = row0 + (int)(blockIdx.x / n);
  const TkGroup gr = (kSuper ? tk.sgroups : tk.groups)[gi];
  if constexpr (kSuper) {
    uint32_t* dst = tk.sghist + ((int64_t)row * tk.n_sgroups + gi) * kTkHistPad;
    for (int b = threadIdx.x; b < kTkHistPad; b += kBlock) {
      uint32_t acc = 0;
      const uint32_t* src = tk.ghist + ((int64_t)row * tk.n_groups + gr.first) * kTkHistPad + b;
#pragma unroll 8
      for (int i = 0; i < gr.n; ++i) acc += src[(int64_t)i * kTkHistPad];
      dst[b] = acc;
    }
  } else {
    __shared__ uint32_t h[kTkHistPad];
    constexpr int kPer = kTkGroup / kWaves;  // tiles per wave
    static_assert(kPer * kTkTileElems < 65536, "packed 16-bit sums");
    const int lane = lane_id();
    uint32_t v[2];
    tile_hist_sum<kPer>(tk, lay, row, gr.first + wave_id() * kPer,
                        min(kPer, gr.n - wave_id() * kPer), lane, v);
    for (int i = threadIdx.x; i < kTkHistPad; i += kBlock) h[i] = 0;
    lds_barrier();
    tile_hist_add(h, lane, v);
    lds_barrier();
    uint32_t* dst = tk.ghist + ((int64_t)row * tk.n_groups + gi) * kTkHistPad;
    for (int i = threadIdx.x; i < kTkHistPad; i += kBlock) dst[i] = h[i];
  }
}

// ------------------------------------------------------------------ block helpers
// Exclusive prefix sum of v over the workgroup (threads in order); *total
// receives the sum.  s must hold blockDim.x / 64 entries.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* s, uint32_t* total) {
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  const int nwaves = blockDim.x / kWave;
  uint32_t x = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
  if (lane == kWave - 1) s[wave] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
  for (int i = 0; i < nwaves; ++i) {
    if (i < wave) before += s[i];
    all += s[i];
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

// Over the LDS histogram h[0..nb), the bin that holds the need-th element
// counted from the top (kTop) or from the bottom (1 <= need <= total).
// Returns to every thread the bin, how many to take inside it and its count.
template <bool kTop>
__device__ __forceinline__ void find_bin(const uint32_t* h, int nb, int64_t need,
                                         uint32_t* s_scan, uint32_t* s_res, uint32_t& bin,
                                         int64_t& left, uint32_t& count) {
  const int per = (nb + (int)blockDim.x - 1) / (int)blockDim.x;
  if (threadIdx.x == 0) {  // defined result even if need exceeded the total
    s_res[0] = 0;
    s_res[1] = 1;
    s_res[2] = 0;
  }
  // thread t owns positions [t per, (t+1) per) counted in the search direction
  uint32_t tot = 0;
  for (int j = 0; j < per; ++j) {
    const int q = threadIdx.x * per + j;
    if (q < nb) tot += h[kTop ? nb - 1 - q : q];
  }
  uint32_t all;
  const uint32_t before = block_excl_scan(tot, s_scan, &all);
  if ((int64_t)before < need && need <= (int64_t)before + tot) {
    int64_t run = before;
    for (int j = 0; j < per; ++j) {
      const int q = threadIdx.x * per + j;
      if (q >= nb) break;
      const int b = kTop ? nb - 1 - q : q;
      if (run + h[b] >= need) {
        s_res[0] = (uint32_t)b;
        s_res[1] = (uint32_t)(need - run);
        s_res[2] = h[b];
        break;
      }
      run += h[b];
    }
  }
  __syncthreads();
  bin = s_res[0];
  left = s_res[1];
  count = s_res[2];
  __syncthreads();
}

// ------------------------------------------------------------------ selection
// The selection of a (row, tensor): the bin b1 of the summed histograms that
// holds the k-th largest key gives the key range [lo, up) of the candidates;
// elements above it are kept for sure, and among the candidates the `need`
// first by (key descending, index ascending) are.  The threshold tau and the
// last kept index iota among the keys equal to it describe the kept set, and
// each tile's first rank follows from its counts.  The order in which
// candidates are collected does not matter.
constexpr int kPick = 256;      // threads of the pick
constexpr int kPickWide = 1024;  // or this many (kTkPickTiles, kTkWidePairs)
constexpr int kSelect = 512;    // threads of the select of large tensors
constexpr int kPickCand = 1024;  // candidates the pick keeps in LDS
constexpr int kSelKeys = 4096;  // candidates whose keys the select keeps in LDS
constexpr int kSelTiles = 2048; // tiles whose counts the select's LDS holds (packed 16-bit)
// A bin with more candidates is full and narrowed first: where there is a refine
// anyway (one tensor of 2^24: 440 us per iteration, 478 at 16384), and else
// (resnet50 K = 8 Top-10%: 1054 us, 1118 at 4096).
constexpr int kRefineCand = 4096;
constexpr int kFullCand = 16384;
constexpr int kRefineLevels = kTkRefineLevels;
constexpr int kGatherSplit = kTkGatherSplit;
constexpr int kGatherTiles = kTkGroup / kGatherSplit;  // tiles per gather workgroup
constexpr int kGatherWide = kGatherTiles * kWave;      // a wave per tile
static_assert(kTkTileElems < 65536 / 2, "a tile's counts fit 16 bits");

// The smallest key of bin b for the near range at win (hist_bin's layout; a
// bin below key 0 is empty and starts at 0); kTkHist (one past the last bin)
// gives 2^31, above every key.
__device__ __forceinline__ uint32_t bin_floor(uint32_t b, uint32_t win) {
  if (b >= (uint32_t)kTkHist) return 0x80000000u;
  int64_t f;
  if (b < (uint32_t)kTkBelow) {
    // bin g of the side: distances up to (below) the first of bin g + 1
    const int64_t g = kTkBelow - 1 - (int64_t)b;
    if (g == kTkBelow - 1) return 0u;
    f = (int64_t)win - (g < kTkMidB ? (g + 1) << kTkMidShift
                                    : (g - kTkMidB + kMidFarB + 1) << kTkFarShift);
  } else if (b < (uint32_t)(kTkBelow + kTkNear)) {
    f = (int64_t)win + ((int64_t)(b - kTkBelow) << kTkSubShift);
  } else {
    const int64_t g = (int64_t)b - (kTkBelow + kTkNear);
    f = (int64_t)win + ((int64_t)kTkNear << kTkSubShift) +
        (g <= kTkMidA ? g << kTkMidShift : (g - kTkMidA + kMidFarA) << kTkFarShift);
  }
  return f <= 0 ? 0u : f < 0x80000000ll ? (uint32_t)f : 0x80000000u;
}

// Bits of the indexes 0 .. n - 1 (1 <= n <= 2^28).
__device__ __forceinline__ int index_bits(int64_t n) {
  return n > 1 ? 32 - __builtin_clz((uint32_t)(n - 1)) : 0;
}

// Bits of the offsets 0 .. up - lo - 1 of the keys in [lo, up).
__device__ __forceinline__ int range_bits(uint32_t lo, uint32_t up) {
  const uint32_t last = up - lo - 1u;
  return up <= lo || last == 0u ? 0 : 32 - __builtin_clz(last);
}

// A candidate: key | (index in the tensor) << 32.
__device__ __forceinline__ u64 cand_of(uint32_t key, int64_t idx) {
  return (u64)key | ((u64)idx << 32);
}

__device__ __forceinline__ void tile_count_add(uint32_t* t, int tile, uint32_t n) {
  atomicAdd(&t[tile >> 1], n << (16 * (tile & 1)));
}
__device__ __forceinline__ uint32_t tile_count(const uint32_t* t, int tile) {
  return (t[tile >> 1] >> (16 * (tile & 1))) & 0xFFFFu;
}

// A tile's 2048 elements of Delta, word by word (lane i: element 64 u + i),
// all loads in flight at once; past the tile's end 0.
__device__ __forceinline__ void load_tile(const float* d, int count, float (&v)[kTileWords]) {
  const Buf r = buf_of(d, (uint32_t)count * 4u);
#pragma unroll
  for (int u = 0; u < kTileWords; ++u)
    v[u] = buf_ld(r, (uint32_t)(u * kWave + lane_id()) * 4u);
}

// The position of the r-th set bit of w (r counted from 0, r < popcount(w)):
// the 32-bit half that holds it, then five halving steps.
__device__ __forceinline__ int nth_set_bit(u64 w, uint32_t r) {
  uint32_t x = (uint32_t)w;
  int pos = 0;
  const uint32_t c_lo = (uint32_t)__popc(x);
  if (r >= c_lo) {
    r -= c_lo;
    x = (uint32_t)(w >> 32);
    pos = 32;
  }
#pragma unroll
  for (int s = 16; s >= 1; s >>= 1) {
    const uint32_t c = (uint32_t)__popc(x & ((1u << s) - 1u));
    if (r >= c) {
      r -= c;
      x >>= s;
      pos += s;
    }
  }
  return pos;
}

// Counts each ok lane's bin into the LDS histogram h.  The server's errors
// crowd a few bins (most of them keep last call's residual, and its binade),
// and one 64-lane LDS atomic into one address is serialized lane by lane: the
// lanes that share the first lane's bin add their count with one atomic, the
// others theirs one by one.  At resnet50 K = 8 Top-1% (union gathers) that
// took the iteration from 0.974-0.977 to 0.965-0.968 ms; repeating it for a
// second bin gave 0.976, a third 0.987-0.990 ms.
__device__ __forceinline__ void hist_add(uint32_t* h, uint32_t bin, bool ok) {
  const int lane = lane_id();
  const u64 todo = __ballot(ok);
  if (todo == 0ull) return;  // wave-uniform
  const int lead = __builtin_ctzll(todo);
  const uint32_t lb = (uint32_t)__builtin_amdgcn_readlane((int)bin, lead);
  const u64 same = __ballot(bin == lb) & todo;
  if (lane == lead)
    atomicAdd(&h[lb], (uint32_t)__popcll(same));
  else if (((todo & ~same) >> lane) & 1ull)
    atomicAdd(&h[bin], 1u);
}

// Where a wave's candidates go: the LDS buffer lds (in_lds), else glb; both
// filled through the LDS count *fill.
struct CandSink {
  uint32_t* fill;
  u64* lds;
  u64* glb;
  uint32_t cap_lds, cap_glb;
  bool in_lds;

  // Space for `total` candidates of the wave (wave-uniform): the first's place.
  __device__ __forceinline__ uint32_t take(uint32_t total) const {
    uint32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(fill, total);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
  }
  // The lanes of mask m put theirs from place `base` on.
  __device__ __forceinline__ void put(u64 m, uint32_t base, uint32_t key, int64_t idx) const {
    const uint32_t pos =
        base + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if (((m >> lane_id()) & 1ull) == 0ull) return;
    if (in_lds) {
      if (pos < cap_lds) lds[pos] = cand_of(key, idx);  // always holds
    } else if (pos < cap_glb) {                         // always holds
      glb[pos] = cand_of(key, idx);
    }
  }
};

// Of a tile: elements with a key at or above up, and those in [lo, up).
struct TileCounts {
  uint32_t sure, cand;
};

// kT tiles (from tile t0 of the tensor on, those below tend) by one wave:
// the elements in [lo, up) go to the sink; returns in lane j the counts of
// tile t0 + j.  n: lane j holds the tile's list count (kTkSpecNone: no usable
// list; 0 past tend).  Taken from the lists (kC chunks of 64 entries of the
// kT tiles in flight together), else from Delta (kW words' loads in flight),
// and then, with relist, the tile's list is written again down to lo (in index
// order, when it fits), for the emit, which would read Delta once more.
template <int kT, int kC, int kW>
__device__ __forceinline__ TileCounts scan_tiles(const CandSink& sink, const DevLayout& lay,
                                                 const TkDev& tk, const TensorInfo& ten, int row,
                                                 int t0, uint32_t n,
                                                 const float* __restrict__ dr, uint32_t lo,
                                                 uint32_t up, bool relist) {
  static_assert(kTileWords % kW == 0, "whole passes over a tile");
  const int lane = lane_id();
  const int64_t tile0 = (int64_t)row * lay.n_tiles + ten.first_tile + t0;
  const u64 none = __ballot(n == kTkSpecNone);
  uint32_t most = n == kTkSpecNone ? 0u : n;
#pragma unroll
  for (int off = 1; off < kT; off <<= 1) most = max(most, (uint32_t)__shfl_xor((int)most, off));
  most = (uint32_t)__builtin_amdgcn_readfirstlane((int)most);
  uint32_t sure = 0, within = 0;
  const u64* ent = tk.spec + tile0 * kTkSpecCap;
  for (uint32_t c0 = 0; c0 < most; c0 += kC * kWave) {
    u64 e[kT][kC], m[kT][kC];
#pragma unroll
    for (int j = 0; j < kT; ++j) {
      const uint32_t nj = (uint32_t)__builtin_amdgcn_readlane((int)n, j);
#pragma unroll
      for (int c = 0; c < kC; ++c) {
        const uint32_t i = c0 + (uint32_t)(c * kWave + lane);
        // (past the list's end, or without a list, the first tile's first
        // entry: it exists)
        e[j][c] = ent[nj != kTkSpecNone && i < nj ? (uint32_t)j * kTkSpecCap + i : 0u];
      }
    }
    uint32_t total = 0;
#pragma unroll
    for (int j = 0; j < kT; ++j) {
      const uint32_t nj = (uint32_t)__builtin_amdgcn_readlane((int)n, j);
      uint32_t above = 0;
      const uint32_t before = total;
#pragma unroll
      for (int c = 0; c < kC; ++c) {
        const bool ok = nj != kTkSpecNone && c0 + (uint32_t)(c * kWave + lane) < nj;
        const uint32_t key = (uint32_t)e[j][c] & 0x7FFFFFFFu;
        above += (uint32_t)__popcll(__ballot(ok && key >= up));
        m[j][c] = __ballot(ok && key >= lo && key < up);
        total += (uint32_t)__popcll(m[j][c]);
      }
      sure += lane == j ? above : 0u;
      within += lane == j ? total - before : 0u;
    }
    if (total == 0u) continue;  // wave-uniform
    uint32_t base = sink.take(total);
#pragma unroll
    for (int j = 0; j < kT; ++j)
#pragma unroll
      for (int c = 0; c < kC; ++c) {
        if (m[j][c] == 0ull) continue;  // wave-uniform
        sink.put(m[j][c], base, (uint32_t)e[j][c] & 0x7FFFFFFFu,
                 (int64_t)(t0 + j) * kTkTileElems + (int64_t)(e[j][c] >> 32));
        base += (uint32_t)__popcll(m[j][c]);
      }
  }
  for (u64 todo = none; todo != 0ull; todo &= todo - 1ull) {  // wave-uniform
    const int j = __builtin_ctzll(todo);
    const int64_t first = (int64_t)(t0 + j) * kTkTileElems;
    const int count = (int)min((int64_t)kTkTileElems, ten.n - first);
    const Buf rd = buf_of(dr + ten.off + first, (uint32_t)count * 4u);
    uint32_t above = 0, inside = 0, listed = 0;
    u64* list = tk.spec + (tile0 + j) * kTkSpecCap;
    const bool whole = count == kTkTileElems;  // wave-uniform
#pragma unroll 1
    for (int w = 0; w < kTileWords; w += kW) {
      float v[kW];
      u64 m[kW];
#pragma unroll
      for (int u = 0; u < kW; ++u) v[u] = buf_ld(rd, (uint32_t)((w + u) * kWave + lane) * 4u);
      uint32_t total = 0;
#pragma unroll
      for (int u = 0; u < kW; ++u) {
        const uint32_t key = key_of(v[u]);
        u64 gl = __ballot(key >= lo);
        const u64 gu = __ballot(key >= up);
        // past the tile's end the keys are 0: below up, but not below a lo of 0
        if (!whole) gl &= __ballot((w + u) * kWave + lane < count);
        m[u] = gl & ~gu;
        above += (uint32_t)__popcll(gu);
        total += (uint32_t)__popcll(m[u]);
        if (relist && gl != 0ull) {  // wave-uniform
          const uint32_t pos =
              listed + __builtin_amdgcn_mbcnt_hi((uint32_t)(gl >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)gl, 0u));
          if (((gl >> lane) & 1ull) && pos < (uint32_t)kTkSpecCap)
            list[pos] = (u64)__float_as_uint(v[u]) | ((u64)((w + u) * kWave + lane) << 32);
          listed += (uint32_t)__popcll(gl);
        }
      }
      if (total == 0u) continue;  // wave-uniform
      inside += total;
      uint32_t base = sink.take(total);
#pragma unroll
      for (int u = 0; u < kW; ++u) {
        if (m[u] == 0ull) continue;  // wave-uniform
        sink.put(m[u], base, key_of(v[u]), first + (w + u) * kWave + lane);
        base += (uint32_t)__popcll(m[u]);
      }
    }
    if (relist && lane == 0)
      tk.lcnt[tile0 + j] = listed <= (uint32_t)kTkSpecCap ? listed : kTkSpecNone;
    sure += lane == j ? above : 0u;
    within += lane == j ? inside : 0u;
  }
  return TileCounts{sure, within};
}

// Counts (key - lo) >> sh of the elements in [lo, up) of one tile (number tile
// of its tensor, ti in the scratch) into the LDS histogram h, by one wave: from
// its list of n entries, or (kTkSpecNone) from Delta, kW words in flight.
template <int kW>
__device__ __forceinline__ void tile_range_hist(uint32_t* h, const TkDev& tk,
                                                const TensorInfo& ten, int64_t ti, int tile,
                                                uint32_t n, const float* __restrict__ dr,
                                                uint32_t lo, uint32_t up, int sh) {
  const int lane = lane_id();
  if (n != kTkSpecNone) {
    const u64* ent = tk.spec + ti * kTkSpecCap;
    for (uint32_t i0 = 0; i0 < n; i0 += kWave) {
      const uint32_t i = i0 + (uint32_t)lane;
      const uint32_t key = (uint32_t)ent[i < n ? i : 0u] & 0x7FFFFFFFu;
      const bool ok = i < n && key >= lo && key < up;
      hist_add(h, ok ? (key - lo) >> sh : 0u, ok);
    }
    return;
  }
  const int64_t first = (int64_t)tile * kTkTileElems;
  const int count = (int)min((int64_t)kTkTileElems, ten.n - first);
  const Buf rd = buf_of(dr + ten.off + first, (uint32_t)count * 4u);
#pragma unroll 1
  for (int w = 0; w < kTileWords; w += kW) {
    float v[kW];
#pragma unroll
    for (int u = 0; u < kW; ++u) v[u] = buf_ld(rd, (uint32_t)((w + u) * kWave + lane) * 4u);
#pragma unroll
    for (int u = 0; u < kW; ++u) {
      const uint32_t key = key_of(v[u]);
      const bool ok = (w + u) * kWave + lane < count && key >= lo && key < up;
      hist_add(h, ok ? (key - lo) >> sh : 0u, ok);
    }
  }
}

// The candidates of a (row, tensor): n of them at p (LDS, or slots), or, when
// segs is not null, in nseg segments of `stride` slots each, segs[i] of them at
// p + i stride.
struct Cands {
  const u64* p;
  int64_t n;
  const uint32_t* segs;
  int nseg;
  uint32_t stride;

  // f(candidate, whether there is one) over all of them by the workgroup, in
  // wave-uniform flow.
  template <typename F>
  __device__ __forceinline__ void each(F f) const {
    if (segs == nullptr) {
      constexpr int kIlp = 4;
      const int64_t nt = blockDim.x;
      for (int64_t b0 = wave_id() * kWave; b0 < n; b0 += nt * kIlp) {
        const int64_t i0 = b0 + lane_id();
        u64 e[kIlp];
#pragma unroll
        for (int u = 0; u < kIlp; ++u) e[u] = p[i0 + u * nt < n ? i0 + u * nt : 0];
#pragma unroll
        for (int u = 0; u < kIlp; ++u)
          if (b0 + u * nt < n) f(e[u], i0 + u * nt < n);
      }
      return;
    }
    const int nw = (int)blockDim.x / kWave;
    constexpr int kS = 4, kC = 4;  // segments, and chunks of each, in flight
    for (int s0 = wave_id() * kS; s0 < nseg; s0 += nw * kS) {
      uint32_t c[kS], most = 0;
#pragma unroll
      for (int q = 0; q < kS; ++q) {
        c[q] = s0 + q < nseg ? segs[s0 + q] : 0u;
        most = max(most, c[q]);
      }
      most = (uint32_t)__builtin_amdgcn_readfirstlane((int)most);
      for (uint32_t b = 0; b < most; b += kC * kWave) {
        u64 e[kC][kS];
#pragma unroll
        for (int a = 0; a < kC; ++a) {
          const uint32_t i = b + (uint32_t)(a * kWave + lane_id());
#pragma unroll
          for (int q = 0; q < kS; ++q)
            e[a][q] = p[i < c[q] ? (int64_t)(s0 + q) * stride + i : (int64_t)s0 * stride];
        }
#pragma unroll
        for (int a = 0; a < kC; ++a) {
          const uint32_t i = b + (uint32_t)(a * kWave + lane_id());
          if (b + (uint32_t)(a * kWave) >= most) break;  // wave-uniform
#pragma unroll
          for (int q = 0; q < kS; ++q) f(e[a][q], i < c[q]);
        }
      }
    }
  }
};

// One radix pass: histogram of digit(e) of the candidates with match(e).
template <typename Match, typename Dig>
__device__ __forceinline__ void cand_hist(uint32_t* h, int nb, const Cands& cand, Match match,
                                          Dig digit) {
  for (int i = threadIdx.x; i < nb; i += blockDim.x) h[i] = 0;
  __syncthreads();
  cand.each([&](u64 e, bool ok) {
    const bool take = ok && match(e);
    hist_add(h, take ? digit(e) : 0u, take);
  });
  __syncthreads();
}

// The next digit of `open` bits taken in as few, and as even, digits of at
// most `most` bits as possible.
__device__ __forceinline__ int radix_digit(int open, int most) {
  const int passes = (open + most - 1) / most;
  return (open + passes - 1) / passes;
}

// tau and iota of the `need` first of C candidates, all with keys below lo +
// 2^open (need <= C): up to one per thread in LDS (lds) by counting each one's
// rank (one pass, no histogram), else radix passes of at most kDig bits over
// key - lo, and, when only some of the keys equal to tau are kept, over the
// index (idx_bits bits).  keys: the candidates' key - lo in LDS, in any order,
// or null (then every pass reads cand).  Every thread of the workgroup calls it
// and gets the result.  h: 2^kDig bins.
template <int kDig>
__device__ __forceinline__ void cand_select(uint32_t* h, uint32_t* scan, uint32_t* res,
                                            const u64* lds, const uint32_t* keys,
                                            const Cands& cand, int64_t C, int64_t need,
                                            uint32_t lo, int open, int idx_bits,
                                            uint32_t& tau, int64_t& iota) {
  if (lds != nullptr && C <= (int64_t)blockDim.x) {
    if (threadIdx.x == 0) {  // defined result even if need exceeded C
      res[0] = lo;
      res[1] = 0xFFFFFFFFu;
    }
    __syncthreads();
    if ((int64_t)threadIdx.x < C) {
      const u64 me = lds[threadIdx.x];
      // (key, then the lower index first) as one number
      const u64 mine = (me << 32) | (uint32_t)~(uint32_t)(me >> 32);
      int before = 0;  // candidates that come first
#pragma unroll 8
      for (int j = 0; j < (int)C; ++j) {
        const u64 e = lds[j];
        before += ((e << 32) | (uint32_t)~(uint32_t)(e >> 32)) > mine ? 1 : 0;
      }
      if (before == (int)need - 1) {
        res[0] = (uint32_t)me;
        res[1] = (uint32_t)(me >> 32);
      }
    }
    __syncthreads();
    tau = res[0];
    iota = (int64_t)res[1];
    __syncthreads();
    return;
  }
  uint32_t prefix = 0, bin = 0, cnt = (uint32_t)C;
  int64_t left = need;
  while (open > 0) {
    const int d = radix_digit(open, kDig);
    const int sh = open - d;
    const uint32_t mask = (1u << d) - 1u;
    const auto match = [=](uint32_t rel) { return (rel >> open) == prefix; };  // open < 32
    if (keys != nullptr) {
      for (int i = threadIdx.x; i < 1 << d; i += blockDim.x) h[i] = 0;
      __syncthreads();
      for (int b = wave_id() * kWave; b < (int)C; b += (int)blockDim.x) {
        const int i = b + lane_id();
        const uint32_t rel = keys[min(i, (int)C - 1)];
        const bool ok = i < (int)C && match(rel);
        hist_add(h, ok ? (rel >> sh) & mask : 0u, ok);
      }
      __syncthreads();
    } else {
      cand_hist(h, 1 << d, cand, [=](u64 e) { return match((uint32_t)e - lo); },
                [=](u64 e) { return (((uint32_t)e - lo) >> sh) & mask; });
    }
    find_bin<true>(h, 1 << d, need, scan, res, bin, left, cnt);
    prefix = (prefix << d) | bin;
    open = sh;
    need = left;
  }
  tau = lo + prefix;
  iota = INT64_MAX;  // every element equal to tau is kept
  if (left < (int64_t)cnt) {
    // the left-th smallest index among the elements equal to tau
    const uint32_t key = tau;
    uint32_t at = 0;
    open = idx_bits;
    need = left;
    while (open > 0) {
      const int d = radix_digit(open, kDig);
      const int sh = open - d;
      const uint32_t mask = (1u << d) - 1u;
      cand_hist(h, 1 << d, cand,
                [=](u64 e) {
                  return (uint32_t)e == key && ((uint32_t)(e >> 32) >> open) == at;
                },
                [=](u64 e) { return ((uint32_t)(e >> 32) >> sh) & mask; });
      find_bin<false>(h, 1 << d, need, scan, res, bin, left, cnt);
      at = (at << d) | bin;
      open = sh;
      need = left;
    }
    iota = (int64_t)at;
  }
}

__device__ __forceinline__ bool cand_kept(u64 e, uint32_t tau, int64_t iota) {
  const uint32_t key = (uint32_t)e;
  return key > tau || (key == tau && (int64_t)(e >> 32) <= iota);
}

// Adds the kept candidates to the tile counts t in LDS, then writes each
// tile's first rank (the exclusive prefix of the counts) to cnt.
__device__ __forceinline__ void tile_ranks(uint32_t* t, uint32_t* scan, const Cands& cand,
                                           uint32_t tau, int64_t iota, int ntiles,
                                           uint32_t* __restrict__ cnt) {
  cand.each([&](u64 e, bool ok) {
    const uint32_t i = (uint32_t)(e >> 32) / kTkTileElems;
    if (ok && cand_kept(e, tau, iota) && i < (uint32_t)ntiles) tile_count_add(t, (int)i, 1u);
  });
  __syncthreads();
  uint32_t carry = 0;
  for (int b = 0; b < ntiles; b += (int)blockDim.x) {
    const int i = b + (int)threadIdx.x;
    uint32_t all;
    const uint32_t v = i < ntiles ? tile_count(t, i) : 0u;
    const uint32_t before = block_excl_scan(v, scan, &all);  // ends with a barrier
    if (i < ntiles) cnt[i] = carry + before;
    carry += all;
  }
}

// Grid: R * nl workgroups, nl the part's tensors (workgroup b: tensor
// p.l0 + b % nl of row row0 + b / nl).  Adds the tile histograms of a small
// tensor, or a large one's group sums or super-group sums, and finds b1.  A
// small tensor is then selected here as a whole, from its tiles' lists or
// Delta (resnet56 Top-5%: one kernel of 13-24 us for six of 44 us); for a
// large one the candidate range and the number to take are left to refine,
// gather and select.  A bin with more candidates than its LDS holds is narrowed
// first, 11 key bits per pass over the tensor's lists or Delta, until they fit
// or are all equal.  256 threads, so that its workgroups find wave slots beside
// a Delta pass (a select of 1024 threads waited up to 200 us for them, until
// the pass drained), or 1024 (kTkPickTiles, kTkWidePairs).
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_tk_pick(DevLayout lay, TkDev tk, TkPart p,
                                                      int row0, const float* __restrict__ data) {
  constexpr int kDig = 8;
  constexpr int kPW = kThreads / kWave;
  __shared__ uint32_t h[kTkHistPad > (1 << kDig) ? kTkHistPad : (1 << kDig)];
  __shared__ u64 s_cand[kPickCand];
  __shared__ uint32_t s_t[kTkGroup / 2];
  __shared__ uint32_t s_scan[kPW];
  __shared__ uint32_t s_res[3];
  __shared__ uint32_t s_fill;
  const int nl = p.l1 - p.l0;
  const int l = p.l0 + (int)(blockIdx.x % (unsigned)nl);
  const int r = (int)(blockIdx.x / (unsigned)nl);
  const int row = row0 + r;
  const TkTensor t = tk.tens[l];
  const TensorInfo ten = lay.tensors[l];
  TkSel* st = tk.sel + (int64_t)row * lay.L + l;
  const uint32_t win = st->win;
  const uint32_t floor = spec_floor(*st);
  const int lane = lane_id(), wave = wave_id();
  const bool small = t.ngroups == 0;
  for (int i = threadIdx.x; i < kTkHistPad; i += kThreads) h[i] = 0;
  if (threadIdx.x < kTkGroup / 2) s_t[threadIdx.x] = 0;
  if (threadIdx.x == 0) s_fill = 0;
  constexpr int kPer = kThreads == kPick ? 8 : 4;  // tiles a wave has in flight
  const int per = (ten.ntiles + kPW - 1) / kPW;  // a wave's tiles: wave per + 0 .. per - 1
  const int tw0 = wave * per, tend = min(tw0 + per, ten.ntiles);
  // lane j: list count of the wave's tile j
  uint32_t lcnt = 0;
  if (small && tw0 + lane < tend)
    lcnt = tk.lcnt[(int64_t)row * lay.n_tiles + ten.first_tile + tw0 + lane];
  if (small) {
    lds_barrier();
    for (int t0 = tw0; t0 < tend; t0 += kPer) {
      uint32_t v[2];
      const int n = min(kPer, tend - t0);
      if (n == 1)
        tile_hist_sum<1>(tk, lay, row, ten.first_tile + t0, n, lane, v);
      else
        tile_hist_sum<kPer>(tk, lay, row, ten.first_tile + t0, n, lane, v);
      tile_hist_add(h, lane, v);
    }
  } else {
    lds_barrier();
    const bool super = t.nsgroups > 0;
    const uint32_t* src = super
        ? tk.sghist + ((int64_t)row * tk.n_sgroups + t.first_sgroup) * kTkHistPad
        : tk.ghist + ((int64_t)row * tk.n_groups + t.first_group) * kTkHistPad;
    const int ns = super ? t.nsgroups : t.ngroups;
    for (int b = threadIdx.x; b < kTkHistPad; b += kPick) {
      uint32_t cnt = 0;
#pragma unroll 8
      for (int i = 0; i < ns; ++i) cnt += src[(int64_t)i * kTkHistPad + b];
      h[b] = cnt;
    }
  }
  __syncthreads();
  uint32_t b1, n1;
  int64_t need;
  find_bin<true>(h, kTkHist, t.keep, s_scan, s_res, b1, need, n1);
  uint32_t lo = bin_floor(b1, win), up = bin_floor(b1 + 1u, win);
  if (!small) {
    const bool coarse = n1 > (uint32_t)(tk.levels != 0 ? kRefineCand : kFullCand);
    if (coarse) {
      uint32_t* rh = tk.rhist + ((int64_t)row * tk.n_large + t.large) * (kRefineLevels * kTkBins);
      for (int i = threadIdx.x; i < max(tk.levels, 1) * kTkBins; i += kThreads) rh[i] = 0;
    }
    if (threadIdx.x == 0) {
      st->floor = floor;
      st->coarse = coarse ? 1u : 0u;
      st->lo = lo;
      st->up = up;
      st->need = need;
    }
    return;
  }
  const float* dr = data + (int64_t)r * lay.d_pad;
  static_assert(sizeof(s_cand) >= kTkBins * sizeof(uint32_t), "a narrowing histogram fits");
  uint32_t* nh = reinterpret_cast<uint32_t*>(s_cand);
  while (n1 > (uint32_t)kPickCand && range_bits(lo, up) > 0) {  // workgroup-uniform
    const int sh = max(range_bits(lo, up) - 11, 0);
    for (int i = threadIdx.x; i < kTkBins; i += kThreads) nh[i] = 0;
    lds_barrier();
    for (int q = tw0; q < tend; ++q) {
      const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)lcnt, q - tw0);
      tile_range_hist<8>(nh, tk, ten, (int64_t)row * lay.n_tiles + ten.first_tile + q, q,
                         floor <= lo ? n : kTkSpecNone, dr, lo, up, sh);
    }
    lds_barrier();
    uint32_t bin;
    const int64_t want = need;
    find_bin<true>(nh, kTkBins, want, s_scan, s_res, bin, need, n1);  // ends with a barrier
    up = min(up, lo + ((bin + 1u) << sh));
    lo = lo + (bin << sh);
  }
  u64* slots = tk.cand + (int64_t)row * lay.d_pad + ten.off;
  const bool in_lds = n1 <= (uint32_t)kPickCand;
  const CandSink sink{&s_fill, s_cand, slots, kPickCand, (uint32_t)ten.n, in_lds};
  const bool relist = st->lists != 0u;
  if (floor > lo && lane < tend - tw0) lcnt = kTkSpecNone;  // the lists end above b1
  for (int t0 = tw0; t0 < tend; t0 += kPer) {
    const uint32_t n = (uint32_t)__shfl((int)lcnt, (t0 - tw0 + lane) % kWave);
    const TileCounts tc =
        scan_tiles<kPer, 1, 8>(sink, lay, tk, ten, row, t0, lane < kPer ? n : 0u, dr, lo, up,
                               relist);
    if (lane < kPer && t0 + lane < tend) tile_count_add(s_t, t0 + lane, tc.sure);
  }
  __syncthreads();  // candidates in LDS or in the slots, and the tile counts
  const int64_t C = (int64_t)min(s_fill, n1);
  const Cands cand{in_lds ? s_cand : slots, C, nullptr, 0, 0};
  uint32_t tau;
  int64_t iota;
  cand_select<kDig>(h, s_scan, s_res, in_lds ? s_cand : nullptr, nullptr, cand, C, need, lo,
                    range_bits(lo, up), index_bits(ten.n), tau, iota);
  tile_ranks(s_t, s_scan, cand, tau, iota, ten.ntiles,
             tk.tile_cnt + (int64_t)row * lay.n_tiles + ten.first_tile);
  if (threadIdx.x == 0) {
    st->floor = relist ? min(floor, lo) : floor;
    st->tau = tau;
    st->iota = iota;
    st->win = window_for(tau);
  }
}

// Grid: R * n * kGatherSplit workgroups, n the part's groups: workgroup b
// takes kGatherTiles tiles of one group of one row.
struct GatherUnit {
  TkGroup gr;
  int row, part;
  int t0, n;          // first tile in the tensor, tile count (may be <= 0)
  const float* data;  // the row's Delta
};
__device__ __forceinline__ GatherUnit gather_unit(const DevLayout& lay, const TkDev& tk,
                                                  const TkPart& p, int row0,
                                                  const float* __restrict__ data) {
  const unsigned n = (unsigned)(p.g1 - p.g0) * kGatherSplit;
  const unsigned u = blockIdx.x % n;
  const int r = (int)(blockIdx.x / n);
  GatherUnit g;
  g.gr = tk.groups[p.g0 + (int)(u / kGatherSplit)];
  g.row = row0 + r;
  g.part = p.g0 * kGatherSplit + (int)u;
  const int first = (int)(u % kGatherSplit) * kGatherTiles;
  g.t0 = g.gr.first + first - lay.tensors[g.gr.l].first_tile;
  g.n = min(kGatherTiles, g.gr.n - first);
  g.data = data + (int64_t)r * lay.d_pad;
  return g;
}

// The candidate range of a large (row, tensor) and how many to take from it:
// the pick's, narrowed by the first `levels` of the refine's histograms when
// coarse (h: kTkBins entries of LDS).  Every thread of the workgroup calls it.
__device__ __forceinline__ void cand_range(const TkDev& tk, const TkSel& st, int row, int large,
                                           int levels, uint32_t* h, uint32_t* scan, uint32_t* res,
                                           uint32_t& lo, uint32_t& up, int64_t& need) {
  lo = st.lo;
  up = st.up;
  need = st.need;
  if (st.coarse == 0u) return;  // workgroup-uniform
  const uint32_t* rh =
      tk.rhist + ((int64_t)row * tk.n_large + large) * (kRefineLevels * kTkBins);
  for (int v = 0; v < levels; ++v) {
    if (range_bits(lo, up) == 0) return;  // one key (workgroup-uniform)
    for (int i = threadIdx.x; i < kTkBins; i += blockDim.x) h[i] = rh[v * kTkBins + i];
    const int sh = max(range_bits(lo, up) - 11, 0);
    __syncthreads();
    uint32_t bin, cnt;
    const int64_t want = need;
    find_bin<true>(h, kTkBins, want, scan, res, bin, need, cnt);
    up = min(up, lo + ((bin + 1u) << sh));
    lo = lo + (bin << sh);
  }
}

// Counts the top 11 bits of key - lo over [lo, up) of the unit's tiles into the
// LDS histogram h.
__device__ __forceinline__ void unit_range_hist(uint32_t* h, const DevLayout& lay, const TkDev& tk,
                                                const GatherUnit& g, uint32_t floor, uint32_t lo,
                                                uint32_t up) {
  const TensorInfo ten = lay.tensors[g.gr.l];
  const int sh = max(range_bits(lo, up) - 11, 0);
  for (int j = wave_id(); j < g.n; j += (int)blockDim.x / kWave) {
    const int64_t ti = (int64_t)g.row * lay.n_tiles + ten.first_tile + g.t0 + j;
    tile_range_hist<8>(h, tk, ten, ti, g.t0 + j, floor <= lo ? tk.lcnt[ti] : kTkSpecNone, g.data,
                       lo, up, sh);
  }
}

// Adds the LDS histogram h to a level of the (row, large tensor)'s in rhist.
__device__ __forceinline__ void add_range_hist(const uint32_t* h, const TkDev& tk, int row,
                                               int large, int level) {
  uint32_t* rh = tk.rhist + ((int64_t)row * tk.n_large + large) * (kRefineLevels * kTkBins) +
                 level * kTkBins;
  for (int i = threadIdx.x; i < kTkBins; i += blockDim.x)
    if (h[i] != 0u) atomicAdd(&rh[i], h[i]);
}

// A wave's kPer tiles (t0 .. of the tensor, those below tend) to the segment
// that starts at tile seg0: candidates to its slots (filled through the LDS
// count *fill), counts to tile_cnt (and tile_cand).  lcnt: lane j holds the
// list count of tile t0 + j.
template <int kPer, int kC>
__device__ __forceinline__ void gather_tiles(uint32_t* fill, const DevLayout& lay,
                                             const TkDev& tk, const TensorInfo& ten, int row,
                                             int seg0, int t0, int tend, uint32_t lcnt,
                                             uint32_t floor, const float* __restrict__ data,
                                             uint32_t lo, uint32_t up, bool within, bool relist) {
  if (t0 >= tend) return;  // wave-uniform
  u64* slots = tk.cand + (int64_t)row * lay.d_pad + ten.off + (int64_t)seg0 * kTkTileElems;
  const CandSink sink{fill, nullptr, slots, 0, (uint32_t)kGatherTiles * kTkTileElems, false};
  const int lane = lane_id();
  if (floor > lo && lane < min(kPer, tend - t0)) lcnt = kTkSpecNone;  // the lists end above lo
  const TileCounts tc =
      scan_tiles<kPer, kC, 8>(sink, lay, tk, ten, row, t0, lcnt, data, lo, up, relist);
  if (lane < kPer && t0 + lane < tend) {
    const int64_t ti = (int64_t)row * lay.n_tiles + ten.first_tile + t0 + lane;
    tk.tile_cnt[ti] = tc.sure;
    if (within) tk.tile_cand[ti] = tc.cand;
  }
}

// Counts, for the (row, tensor)s whose candidate bin is full, 11 bits of key -
// lo (level 0: the top 11 of the bin's; level 1: the next 11) over the
// candidates of their tiles (from the lists where they reach down to lo, else
// from Delta) in LDS, then adds the bins to rhist; the gather takes the
// sub-range that holds the threshold, mostly one key.  One workgroup's radix
// passes over all the candidates of such a bin (a wide one, or one where
// many values are equal) took up to 3 ms at bert_base Top-1% (K = 16), whose
// outliers all have one magnitude.  Launched for plans with a tensor of more
// than 4096 tiles.  In the others the gather counts and the select's launch
// gathers: launches that mostly find nothing to narrow took resnet50 K = 8 from
// 820 to 825 us per Top-1% iteration and from 1059 to 1077 at Top-10%.
template <int kLevel>
__global__ __launch_bounds__(kBlock) void k_tk_refine(DevLayout lay, TkDev tk, TkPart p, int row0,
                                                      const float* __restrict__ data) {
  __shared__ uint32_t h[kTkBins];
  __shared__ uint32_t s_scan[kWaves];
  __shared__ uint32_t s_res[3];
  const GatherUnit g = gather_unit(lay, tk, p, row0, data);
  const TkSel& st = tk.sel[(int64_t)g.row * lay.L + g.gr.l];
  if (st.coarse == 0u || g.n <= 0) return;  // workgroup-uniform
  const int large = tk.tens[g.gr.l].large;
  const uint32_t floor = st.floor;
  uint32_t lo, up;
  int64_t need;
  cand_range(tk, st, g.row, large, kLevel, h, s_scan, s_res, lo, up, need);
  if (range_bits(lo, up) == 0) return;  // one key already (workgroup-uniform)
  for (int i = threadIdx.x; i < kTkBins; i += kBlock) h[i] = 0;
  lds_barrier();
  unit_range_hist(h, lay, tk, g, floor, lo, up);
  lds_barrier();
  add_range_hist(h, tk, g.row, large, kLevel);
}

// Grid: as k_tk_refine.  Each tile's count of elements with a key at or above
// up to tile_cnt, and the elements in [lo, up) to the workgroup's segment of
// the (row, tensor)'s slots (kGatherTiles tiles' slots: they fit), their
// number to seg.  From the lists where they reach down to lo, else from Delta.
// Of a full bin that no refine narrows (a threshold that moved far) it only
// counts 11 bits of key - lo into rhist; the select's launch gathers.
template <int kC, int kThreads>
__global__ __launch_bounds__(kThreads) void k_tk_gather(DevLayout lay, TkDev tk, TkPart p,
                                                        int row0,
                                                        const float* __restrict__ data) {
  __shared__ uint32_t h[kTkBins];
  __shared__ uint32_t s_scan[kThreads / kWave];
  __shared__ uint32_t s_res[3];
  __shared__ uint32_t s_fill;
  const GatherUnit g = gather_unit(lay, tk, p, row0, data);
  const TensorInfo ten = lay.tensors[g.gr.l];
  uint32_t lo, up;
  int64_t need;
  const TkSel& st = tk.sel[(int64_t)g.row * lay.L + g.gr.l];
  const uint32_t floor = st.floor;
  const int large = tk.tens[g.gr.l].large;
  if (st.coarse != 0u && tk.levels == 0) {  // workgroup-uniform
    if (g.n <= 0) return;
    for (int i = threadIdx.x; i < kTkBins; i += kThreads) h[i] = 0;
    lds_barrier();
    unit_range_hist(h, lay, tk, g, floor, st.lo, st.up);
    lds_barrier();
    add_range_hist(h, tk, g.row, large, 0);
    return;
  }
  constexpr int kPer = kGatherTiles * kWave / kThreads;  // tiles per wave
  const int t0 = g.t0 + wave_id() * kPer, tend = g.t0 + g.n;
  uint32_t lcnt = 0;
  if (lane_id() < kPer && t0 + lane_id() < tend)
    lcnt = tk.lcnt[(int64_t)g.row * lay.n_tiles + ten.first_tile + t0 + lane_id()];
  if (threadIdx.x == 0) s_fill = 0;
  cand_range(tk, st, g.row, large, tk.levels, h, s_scan, s_res, lo, up, need);
  lds_barrier();
  gather_tiles<kPer, kC>(&s_fill, lay, tk, ten, g.row, g.t0, t0, tend, lcnt, floor, g.data, lo, up,
                         tk.levels != 0, st.lists != 0u);
  lds_barrier();
  if (threadIdx.x == 0)
    tk.seg[(int64_t)g.row * tk.n_groups * kGatherSplit + g.part] = s_fill;
}

// The exclusive prefix over the tensor's tiles, in tile order, of f(tile),
// given to put(tile, first, value); eight consecutive tiles per thread.
// Every thread of the workgroup calls it.
template <typename F, typename P>
__device__ __forceinline__ void tile_prefix(int ntiles, uint32_t* scan, F f, P put) {
  constexpr int kQ = 8;
  uint32_t carry = 0;
  for (int b = 0; b < ntiles; b += (int)blockDim.x * kQ) {
    const int i0 = b + (int)threadIdx.x * kQ;
    uint32_t v[kQ], sum = 0;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      v[q] = i0 + q < ntiles ? f(i0 + q) : 0u;
      sum += v[q];
    }
    uint32_t all;
    uint32_t at = carry + block_excl_scan(sum, scan, &all);  // ends with a barrier
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      if (i0 + q < ntiles) put(i0 + q, at, v[q]);
      at += v[q];
    }
    carry += all;
  }
}

// The threshold and tile ranks of a large (row, tensor) from its candidates in
// [lo, up) and tile counts.  When the narrowing left one key, the candidates are
// equal and the first `need` of them by index are kept: the tile counts give the
// tile where they end, and only that tile's candidates are looked at.  Else up to
// kSelTiles tiles are counted in LDS; beyond, in tile_cnt itself with device
// atomics (read back past the L1).
constexpr int kSelDig = 10;
struct SelectLds {
  uint32_t key[kSelKeys];
  uint32_t h[1 << kSelDig];
  uint32_t t[kSelTiles / 2];
  uint32_t scan[kSelect / kWave];
  uint32_t res[3];
  uint32_t fill;
};
static_assert(kSelKeys >= kTkBins, "the range's histogram fits in key");
__device__ __forceinline__ void select_tensor(SelectLds& s, const DevLayout& lay, const TkDev& tk,
                                              const TensorInfo& ten, const TkTensor& t, TkSel* st,
                                              int row, uint32_t lo, uint32_t up, int64_t need) {
  const u64* slots = tk.cand + (int64_t)row * lay.d_pad + ten.off;
  const int64_t tile0 = (int64_t)row * lay.n_tiles + ten.first_tile;
  uint32_t* cnt = tk.tile_cnt + tile0;
  const uint32_t* segs = tk.seg + ((int64_t)row * tk.n_groups + t.first_group) * kGatherSplit;
  const int nseg = t.ngroups * kGatherSplit;
  constexpr uint32_t kStride = (uint32_t)kGatherTiles * kTkTileElems;
  uint32_t tau;
  int64_t iota;
  if (st->coarse != 0u && range_bits(lo, up) == 0) {  // workgroup-uniform
    const uint32_t* within = tk.tile_cand + tile0;
    if (threadIdx.x == 0) {
      s.res[0] = 0;
      s.res[1] = 0;
      s.res[2] = kTkTileElems - 1;
    }
    if (threadIdx.x < kTkTileElems / 32) s.h[threadIdx.x] = 0;
    __syncthreads();
    tile_prefix(ten.ntiles, s.scan, [=](int i) { return within[i]; },
                [&](int i, uint32_t at, uint32_t v) {
                  if ((int64_t)at < need && need <= (int64_t)at + v) {
                    s.res[0] = (uint32_t)i;            // the tile with the last one kept
                    s.res[1] = (uint32_t)(need - at);  // how many of it are kept
                  }
                });
    __syncthreads();
    const int last = (int)s.res[0];
    const uint32_t take = s.res[1];
    // the tile's candidates as bits, then the take-th of them
    const u64* seg = slots + (int64_t)(last / kGatherTiles) * kStride;
    const uint32_t n = min(segs[last / kGatherTiles], kStride);
    for (uint32_t i = threadIdx.x; i < n; i += kSelect) {
      const uint32_t idx = (uint32_t)(seg[i] >> 32);
      if (idx / kTkTileElems == (uint32_t)last)
        atomicOr(&s.h[idx % kTkTileElems / 32], 1u << (idx % 32u));
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
      const uint32_t w = s.h[threadIdx.x];
      const uint32_t c = (uint32_t)__popc(w);
      uint32_t incl = c;
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off);
        if (lane_id() >= off) incl += y;
      }
      static_assert(kTkTileElems == 32 * kWave, "a lane per word of the tile's bits");
      if (incl - c < take && take <= incl)
        s.res[2] = threadIdx.x * 32u + (uint32_t)nth_set_bit((u64)w, take - (incl - c) - 1u);
    }
    __syncthreads();
    tau = lo;
    iota = (int64_t)last * kTkTileElems + s.res[2];
    tile_prefix(ten.ntiles, s.scan,
                [=](int i) { return cnt[i] + (i < last ? within[i] : i == last ? take : 0u); },
                [=](int i, uint32_t at, uint32_t) { cnt[i] = at; });
  } else {
    const bool counted = ten.ntiles <= kSelTiles;
    if (counted)
      for (int i = threadIdx.x; 2 * i < ten.ntiles; i += kSelect)
        s.t[i] = cnt[2 * i] | (2 * i + 1 < ten.ntiles ? cnt[2 * i + 1] << 16 : 0u);
    if (threadIdx.x == 0) s.fill = 0;
    // the number of candidates; the keys of up to kSelKeys are brought to LDS
    uint32_t mine = 0;
    for (int i = threadIdx.x; i < nseg; i += kSelect) mine += segs[i];
    uint32_t total;
    (void)block_excl_scan(mine, s.scan, &total);  // ends with a barrier
    const bool in_lds = total <= (uint32_t)kSelKeys;
    const Cands cand{slots, (int64_t)total, segs, nseg, kStride};
    if (in_lds) {
      cand.each([&](u64 e, bool ok) {
        const u64 m = __ballot(ok);
        if (m == 0ull) return;
        uint32_t base = 0;
        if (lane_id() == 0) base = atomicAdd(&s.fill, (uint32_t)__popcll(m));
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        const uint32_t pos =
            base + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (ok && pos < (uint32_t)kSelKeys) s.key[pos] = (uint32_t)e - lo;  // always holds
      });
      __syncthreads();
    }
    cand_select<kSelDig>(s.h, s.scan, s.res, nullptr, in_lds ? s.key : nullptr, cand,
                         (int64_t)total, need, lo, range_bits(lo, up), index_bits(ten.n), tau,
                         iota);
    if (counted) {
      tile_ranks(s.t, s.scan, cand, tau, iota, ten.ntiles, cnt);
    } else {
      cand.each([&](u64 e, bool ok) {
        const uint32_t i = (uint32_t)(e >> 32) / kTkTileElems;
        if (ok && cand_kept(e, tau, iota) && i < (uint32_t)ten.ntiles) atomicAdd(&cnt[i], 1u);
      });
      __threadfence();
      __syncthreads();
      tile_prefix(ten.ntiles, s.scan,
                  [=](int i) {
                    return __hip_atomic_load(&cnt[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                  },
                  [=](int i, uint32_t at, uint32_t) { cnt[i] = at; });
    }
  }
  __syncthreads();  // every thread has read st
  if (threadIdx.x == 0) {
    if (st->lists != 0u) st->floor = min(st->floor, lo);  // as the gather left the lists
    st->tau = tau;
    st->iota = iota;
    st->win = window_for(tau);
  }
}

// Grid: R * (n + m kParts) workgroups, n the part's large tensors and m its tile
// groups.  Workgroup b < R n: the threshold and tile ranks of large tensor p.b0 +
// b % n of row row0 + b / n from the gathered candidates and counts.  The others
// take a part of a group each and return at once, unless the tensor's candidate
// bin is full and the gather only counted it: then they gather its tiles from
// the sub-range that the counts leave, and the last one of the tensor to arrive
// (nobody waits) selects.  (One workgroup takes up to 4 ms over a full bin:
// resnet50 K = 8 Top-1%, all values 1000 times as large as in the call before,
// 4.4 ms a call; 1.36 ms this way.)
template <int kParts>
__global__ __launch_bounds__(kSelect) void k_tk_select(DevLayout lay, TkDev tk, TkPart p, int R,
                                                       int row0,
                                                       const float* __restrict__ data) {
  constexpr int kSW = kSelect / kWave;
  __shared__ SelectLds s;
  __shared__ uint32_t s_segs[kGatherSplit];
  const unsigned nb = (unsigned)(p.b1 - p.b0), nsel = nb * (unsigned)R;
  const bool helps = blockIdx.x >= nsel;  // workgroup-uniform, like all of this
  int l, lg, row, gi = 0, part = 0;
  if (helps) {
    const unsigned n = (unsigned)(p.g1 - p.g0) * kParts, u = blockIdx.x - nsel;
    gi = p.g0 + (int)(u % n / kParts);
    part = (int)(u % kParts);
    row = row0 + (int)(u / n);
    l = tk.groups[gi].l;
    lg = tk.tens[l].large;
  } else {
    lg = p.b0 + (int)(blockIdx.x % nb);
    row = row0 + (int)(blockIdx.x / nb);
    l = tk.large[lg];
  }
  TkSel* st = tk.sel + (int64_t)row * lay.L + l;
  const TensorInfo ten = lay.tensors[l];
  const TkTensor t = tk.tens[l];
  const TkSel was = *st;
  __builtin_amdgcn_sched_barrier(0);  // these loads before the branch
  const bool full = was.coarse != 0u && tk.levels == 0;
  if (helps != full) return;
  const int levels = full ? 1 : tk.levels;
  uint32_t lo, up;
  int64_t need;
  cand_range(tk, was, row, lg, levels, s.key, s.scan, s.res, lo, up, need);
  if (full) {
    constexpr int kUnit = kTkGroup / kParts, kSegs = kGatherSplit / kParts;
    constexpr int kPer = kUnit / kSW < 4 ? kUnit / kSW : 4, kTurns = kUnit / kSW / kPer;
    static_assert(kGatherTiles % kPer == 0, "the tiles of a turn lie in one segment");
    const TkGroup gr = tk.groups[gi];
    const int g0 = gr.first - ten.first_tile, u0 = g0 + part * kUnit;
    const int tend = min(g0 + gr.n, u0 + kUnit);
    if (threadIdx.x < kSegs) s_segs[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll 1
    for (int q = 0; q < kTurns; ++q) {
      const int t0 = u0 + (wave_id() * kTurns + q) * kPer, seg = (t0 - u0) / kGatherTiles;
      uint32_t lcnt = 0;
      if (lane_id() < kPer && t0 + lane_id() < tend)
        lcnt = tk.lcnt[(int64_t)row * lay.n_tiles + ten.first_tile + t0 + lane_id()];
      gather_tiles<kPer, 1>(&s_segs[seg], lay, tk, ten, row, u0 + seg * kGatherTiles, t0, tend,
                            lcnt, st->floor, data + (int64_t)(row - row0) * lay.d_pad, lo, up, true,
                            st->lists != 0u);
    }
    __syncthreads();
    if (threadIdx.x < kSegs)
      tk.seg[((int64_t)row * tk.n_groups + gi) * kGatherSplit + part * kSegs + threadIdx.x] =
          s_segs[threadIdx.x];
    // Every wave's stores have reached the L2 before the barrier, which does not
    // wait for them by itself; one thread then has the L2 written back for the
    // other XCDs (each release writes back a whole L2: not one per wave), waits
    // for that and arrives.  The last to arrive drops what its caches may hold
    // of the others' results.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t* arrived = tk.arrived + (int64_t)row * tk.n_large + lg;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __builtin_amdgcn_s_waitcnt(0);
      const bool last = atomicAdd(arrived, 1u) + 1u == (uint32_t)(t.ngroups * kParts);
      if (last) atomicExch(arrived, 0u);  // for the next call
      s.res[0] = last ? 1u : 0u;
    }
    __syncthreads();
    if (s.res[0] == 0u) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  select_tensor(s, lay, tk, ten, t, st, row, lo, up, need);
}

// ------------------------------------------------------------------ emit
// A tile's selection words from lane u's word `mine` (u < nw), and its rank
// words: the tile's first rank and the counts of the words before.  Returns
// the lane's word's rank in the tile.
__device__ __forceinline__ uint32_t emit_words(u64 mine, int nw, uint32_t base,
                                               uint64_t* __restrict__ sr,
                                               uint32_t* __restrict__ rr) {
  const int lane = lane_id();
  const uint32_t cnt = (uint32_t)__popcll(mine);
  uint32_t incl = cnt;
#pragma unroll
  for (int off = 1; off < kTileWords; off <<= 1) {
    const uint32_t y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  if (lane < nw) {
    sr[lane] = mine;
    rr[lane] = base + incl - cnt;
  }
  return incl - cnt;
}

// The emit of a tile from its speculative list (n <= 64 kNC entries, index
// order): if the list reaches down to the threshold, an entry is kept iff its
// key is above tau, or equal to it with an index up to iota; its value (from
// the entry) goes to the message at the tile's first rank plus the kept
// entries before it, the error there is set to 0, and the selection words
// (assembled in LDS) and rank words are written.  Returns false, having
// written nothing, otherwise.  The list loads are issued before the selection
// state is waited for.
template <int kNC, bool kX, bool kPend>
__device__ __forceinline__ bool emit_list(const u64* __restrict__ ent, uint32_t n,
                                          const TkSel* stp, int64_t rel0, uint32_t base,
                                          uint32_t keep, int count, int nw,
                                          uint64_t* __restrict__ sr, uint32_t* __restrict__ rr,
                                          float* __restrict__ vr, float* __restrict__ dr,
                                          float* __restrict__ xt, u64* s_w) {
  const int lane = lane_id();
  u64 e[kNC > 0 ? kNC : 1];
#pragma unroll
  for (int c = 0; c < kNC; ++c) {
    const uint32_t i = (uint32_t)(c * kWave + lane);
    e[c] = ent[i < n ? i : 0u];
  }
  const uint32_t tau = stp->tau;
  const int64_t iota = stp->iota;
  if (stp->floor > tau) return false;
  if (lane < kTileWords) s_w[lane] = 0ull;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  uint32_t run = 0;  // kept entries in the earlier chunks
#pragma unroll
  for (int c = 0; c < kNC; ++c) {
    const bool ok = (uint32_t)(c * kWave + lane) < n;
    const uint32_t raw = (uint32_t)e[c], key = raw & 0x7FFFFFFFu;
    const uint32_t idx = (uint32_t)(e[c] >> 32);  // index in the tile
    const bool kept = ok && (key > tau || (key == tau && rel0 + (int64_t)idx <= iota));
    const u64 km = __ballot(kept);
    if (kept) {
      atomicOr(&s_w[idx >> 6], 1ull << (idx & 63u));
      const uint32_t pos = base + run + __builtin_amdgcn_mbcnt_hi((uint32_t)(km >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
      if (pos < keep && idx < (uint32_t)count) {  // both always hold
        vr[pos] = __uint_as_float(raw);
        if (!kPend) st_nt(dr + idx, 0.0f);  // e = Delta - C(Delta) = 0 at a kept element
        if (kX) xt[idx] -= __uint_as_float(raw);
      }
    }
    run += (uint32_t)__popcll(km);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  emit_words(lane < nw ? s_w[lane] : 0ull, nw, base, sr, rr);
  return true;
}

// Grid: ceil((p.t1 - p.t0) / 4) * R workgroups; wave w of workgroup b owns
// tile p.t0 + 4 (b / R) + w of row b % R.  Writes the tile's selection words,
// rank words and kept values in index order, and sets the kept elements of
// data to 0 (kPend: left for the next reader); kX (server): x <- x - Delta at
// the kept elements (C(Delta) is zero elsewhere).  From the tile's list where
// there is one that reaches down to the threshold, else from Delta (one
// streaming read, all 32 words in flight at once).
template <bool kX, bool kPend>
__global__ __launch_bounds__(kBlock) void k_tk_emit(DevLayout lay, TkDev tk, TkPart p, int R,
                                                    int row0, float* __restrict__ data,
                                                    uint64_t* __restrict__ sel,
                                                    uint32_t* __restrict__ rank,
                                                    float* __restrict__ vals,
                                                    float* __restrict__ x) {
  __shared__ u64 words[kWaves][kTileWords];  // one row per wave, used by that wave only
  const int r = (int)(blockIdx.x % (unsigned)R);
  const int64_t ti = p.t0 + (int64_t)(blockIdx.x / (unsigned)R) * kWaves + wave_id();
  if (ti >= p.t1) return;
  const int wave = threadIdx.x / kWave;
  const int lane = lane_id();
  const int row = row0 + r;
  const int64_t rt = (int64_t)row * lay.n_tiles + ti;
  const uint32_t n = tk.lcnt[rt];
  const uint32_t base = tk.tile_cnt[rt];
  const Tile tile = lay.tiles[ti];
  const int nw = (tile.count + 63) >> 6;
  const TkSel* stp = tk.sel + (int64_t)row * lay.L + tile.l;
  const int64_t rel0 = tile.start - lay.tensors[tile.l].off;
  const TkTensor* tp = tk.tens + tile.l;
  const int64_t wat = (int64_t)r * (lay.d_pad >> 6) + (tile.start >> 6);
  uint64_t* sr = sel + wat;
  uint32_t* rr = rank + wat;
  float* vr = vals + (int64_t)r * tk.total_keep + tp->voff;
  float* dr = data + (int64_t)r * lay.d_pad + tile.start;
  const uint32_t keep = (uint32_t)tp->keep;
  float* xt = kX ? x + tile.start : nullptr;
  if (n != kTkSpecNone) {
    static_assert(kTkSpecCap == 8 * kWave, "lists of up to 8 loads per lane");
    const u64* ent = tk.spec + rt * kTkSpecCap;
    bool done;
#define SAEF_EL(NC)                                                                           \
  done = emit_list<NC, kX, kPend>(ent, n, stp, rel0, base, keep, tile.count, nw, sr, rr, vr, \
                                  dr, xt, words[wave])
    switch ((n + kWave - 1) / kWave) {
      case 0: SAEF_EL(0); break;
      case 1: SAEF_EL(1); break;
      case 2: SAEF_EL(2); break;
      case 3: SAEF_EL(3); break;
      case 4: SAEF_EL(4); break;
      case 5: SAEF_EL(5); break;
      case 6: SAEF_EL(6); break;
      case 7: SAEF_EL(7); break;
      default: SAEF_EL(8); break;
    }
#undef SAEF_EL
    if (done) return;
  }
  float v[kTileWords];
  load_tile(dr, tile.count, v);
  const uint32_t tau = stp->tau;
  const int64_t iota = stp->iota;
  // the last kept element equal to tau, in the tile (none: -1; past the tile's
  // end the keys are 0, and kept ones end before it)
  const int last = (int)max((int64_t)-1, min(iota - rel0, (int64_t)tile.count - 1));
  u64 mine = 0;  // lane u: word u
#pragma unroll
  for (int u = 0; u < kTileWords; ++u) {
    const uint32_t key = key_of(v[u]);
    const u64 word = __ballot(key > tau || (key == tau && u * kWave + lane <= last));
    if (lane == u) mine = word;
  }
  const uint32_t excl = emit_words(mine, nw, base, sr, rr);
#pragma unroll
  for (int u = 0; u < kTileWords; ++u) {
    const u64 word = word_of(mine, u);
    if (word == 0ull) continue;  // wave-uniform
    const uint32_t pos =
        base + (uint32_t)__builtin_amdgcn_readlane((int)excl, u) +
        __builtin_amdgcn_mbcnt_hi((uint32_t)(word >> 32),
                                  __builtin_amdgcn_mbcnt_lo((uint32_t)word, 0u));
    const int j = u * kWave + lane;
    if (((word >> lane) & 1ull) && pos < keep) {  // the last always holds
      vr[pos] = v[u];
      if (!kPend) st_nt(dr + j, 0.0f);  // e = Delta - C(Delta) = 0 at a kept element
      if (kX) xt[j] -= v[u];
    }
  }
}

// ------------------------------------------------------------------ server aggregation
// A wave takes whole tiles of a chunk, U selection words (U x 64 elements)
// per pass in word order, and the workers in batches of kWave / U: in a
// batch, lane q loads selection word q % U of worker q / U together with its
// rank word (one vector load each).  The values are gathered per pair (their
// masks and ranks read out of those lanes with v_readlane), per worker for
// dense messages, or over the union of the workers' kept elements (below).
// The words of the next step are loaded before the values of the current one
// are waited for, so one step costs one memory round trip.  The K values of
// an element are added in binary64 in worker order (/K, fp32); mode 1: Delta
// = e_srv + mean stored into e_srv, its pass-1 histogram and the server row's
// speculative lists; mode 0: x <- x - mean.

// A lane's (worker, word) pair: selection word, 4 x rank word (0 for a pair
// that does not exist).
struct AggWords {
  uint32_t lo, hi, rk4;
};
// The pair as loaded, with whether it exists: the words are cleared where
// they are used, in the next step (selects right after the loads made the
// compiler branch around them and wait for them, and so for every load
// issued before them, at once).
struct AggStep {
  u64 s;
  uint32_t r;
  bool ok;
  __device__ __forceinline__ AggWords words() const {
    AggWords a;
    a.lo = ok ? (uint32_t)s : 0u;
    a.hi = ok ? (uint32_t)(s >> 32) : 0u;
    a.rk4 = ok ? r * 4u : 0u;
    return a;
  }
};

template <int U>
__device__ __forceinline__ AggStep agg_words(const uint64_t* __restrict__ sel,
                                             const uint32_t* __restrict__ rank, int64_t W,
                                             int64_t gw, int K, int nw, int w0, int k0,
                                             int lane) {
  const int kq = k0 + lane / U, uq = lane % U;
  AggStep a;
  a.ok = kq < K && w0 + uq < nw;
  // always issued at a word that exists (the chunk's first word of worker 0)
  const int64_t at = a.ok ? (int64_t)kq * W + gw + w0 + uq : gw;
  a.s = sel[at];
  a.r = rank[at];
  return a;
}

// How a pass gathers the K messages' values: per (worker, word) pair, one
// load per worker for dense messages, or over the pass's union (below).
constexpr int kTkAggPairs = 0;
constexpr int kTkAggDense = 1;
constexpr int kTkAggUnion = 2;

// The means of a pass of U words when one batch holds every worker (K <= kWave
// / U; lane q holds the words of worker q / U, word q % U): the elements that
// some worker kept (the union of the K selection words of each word) are
// taken 64 at a time, one per lane, and each lane gathers its element's K
// values (a worker that did not keep it reads past the end of its buffer and
// gets 0), so a sparse pass costs K loads per 64 union elements instead of
// one per (worker, word) pair.  The sum runs over all kWave / U workers in
// order in binary64 (absent ones add +0), as in the per-pair gathers, so the
// means are the same bits.  mb (U x 64 floats, the wave's own) returns them
// per element; an element no worker kept has mean +0.  The wave's pairs go
// to wt (64 entries of 16 bytes) and its union words to ut (U entries): a
// lane reads the entry it needs with one LDS load (lanes of one word read
// one address, and the U entries of a worker are one 16 U-byte span, so the
// loads have no bank conflicts), which keeps the pass off the LDS issue
// limit that one ds_bpermute per word and worker ran into.
template <int U>
__device__ __forceinline__ void union_means(const AggWords& cur, int K, double inv_k,
                                            const float* __restrict__ vals, int64_t total_keep,
                                            uint32_t keep, int lane, float* __restrict__ mb,
                                            uint4* __restrict__ wt, uint4* __restrict__ ut,
                                            float (&mean)[U]) {
  constexpr int kB = kWave / U;
#pragma unroll
  for (int i = 0; i < U; ++i) mb[i * kWave + lane] = 0.0f;
  wt[lane] = make_uint4(cur.lo, cur.hi, cur.rk4, 0u);
  // the union of word q % U in every lane q (absent workers hold empty words)
  uint32_t ulo = cur.lo, uhi = cur.hi;
#pragma unroll
  for (int off = U; off < kWave; off <<= 1) {
    ulo |= (uint32_t)__shfl_xor((int)ulo, off);
    uhi |= (uint32_t)__shfl_xor((int)uhi, off);
  }
  // inclusive scan of the union counts over the U words (every group of U
  // lanes holds the same counts and scans them alike)
  const uint32_t cnt = (uint32_t)(__popc(ulo) + __popc(uhi));
  uint32_t incl = cnt;
#pragma unroll
  for (int off = 1; off < U; off <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)incl, off);
    if ((lane % U) >= off) incl += y;
  }
  if (lane < U) ut[lane] = make_uint4(ulo, uhi, incl - cnt, 0u);
  // the inclusive counts of words 0 .. U - 2, and the pass's union size
  uint32_t inc_s[U - 1];
#pragma unroll
  for (int w = 0; w < U - 1; ++w) inc_s[w] = (uint32_t)__builtin_amdgcn_readlane((int)incl, w);
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, U - 1);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  for (uint32_t i0 = 0; i0 < total; i0 += kWave) {
    const uint32_t i = i0 + (uint32_t)lane;  // the i-th union element of the pass
    // its word: the number of words whose inclusive count is <= i (at most
    // U - 1, for lanes past the end, which load and store nothing)
    int u = 0;
#pragma unroll
    for (int w = 0; w < U - 1; ++w) u += inc_s[w] <= i ? 1 : 0;
    const uint4 uw = ut[u];  // union word, union elements before it
    const int b = nth_set_bit(((u64)uw.y << 32) | uw.x, i - uw.z);
    const bool live = i < total;
    const u64 below_mask = (1ull << b) - 1ull;
    float v[kB];
#pragma unroll
    for (int kk = 0; kk < kB; ++kk) {
      const int kidx = min(kk, K - 1);  // absent workers have empty words
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(vals + (int64_t)kidx * total_keep), 0, (int)(keep * 4u), kBufWord3);
      const uint4 pw = wt[kk * U + u];  // worker kk's selection word, 4 x rank word
      const u64 w = ((u64)pw.y << 32) | pw.x;
      const bool bit = live && ((w >> b) & 1ull) != 0ull;
      const uint32_t off = bit ? pw.z + 4u * (uint32_t)__popcll(w & below_mask) : 0x80000000u;
      v[kk] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
    }
    double acc = 0.0;
#pragma unroll
    for (int kk = 0; kk < kB; ++kk) acc += (double)v[kk];  // worker order; absent: +0
    if (live) mb[u * kWave + b] = (float)mean_of(acc, inv_k, K);
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
  for (int i = 0; i < U; ++i) mean[i] = mb[i * kWave + lane];
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

template <int kMode, bool kAvg, int U, int kPath>
__global__ __launch_bounds__(kAgg) void k_tk_aggregate(DevLayout lay, TkDev tk, TkPart p,
                                                       int K, double inv_k,
                                                       const uint64_t* __restrict__ sel,
                                                       const uint32_t* __restrict__ rank,
                                                       const float* __restrict__ vals,
                                                       float* __restrict__ avg,
                                                       float* __restrict__ es,
                                                       float* __restrict__ x) {
  constexpr int kB = kWave / U;  // workers per batch
  static_assert(kB * U == kWave, "one (worker, word) pair per lane");
  static_assert(kTileWords % U == 0, "a pass of U words stays in one tile");
  constexpr int kChunkTiles = kTkChunk / kTkTileElems;
  __shared__ uint32_t h[kMode == 1 ? kChunkTiles * kTkHistPad : 1];  // per tile of the chunk
  __shared__ float mb[kPath == kTkAggUnion ? (kAgg / kWave) * U * kWave : 1];  // a pass's means
  __shared__ uint4 wt[kPath == kTkAggUnion ? kAgg : 1];                 // per wave: its 64 pairs
  __shared__ uint4 ut[kPath == kTkAggUnion ? (kAgg / kWave) * U : 1];   // per wave: union words
  static_assert(kPath != kTkAggUnion || U * kWave <= (int)(sizeof(mb) / sizeof(float)),
                "a wave's means");
  const int64_t ci = p.c0 + (int64_t)blockIdx.x;
  const TkChunk c = tk.chunks[ci];
  const int64_t voff = tk.tens[c.l].voff;
  const uint32_t keep = (uint32_t)tk.tens[c.l].keep;
  const TkSel* sst = tk.sel + (int64_t)lay.k_max * lay.L + c.l;  // the server row's state
  const uint32_t win = kMode == 1 ? sst->win : 0u;
  // the server row's speculative lists, as the worker Delta pass writes them:
  // per tile, the elements whose key is at least spec_floor, in index order
  const uint32_t lo_spec = kMode == 1 ? spec_floor(*sst) : 0x80000000u;
  const TensorInfo ten = lay.tensors[c.l];
  const int64_t tile0 = ten.first_tile + (c.start - ten.off) / kTkTileElems;
  if (kMode == 1) {
    for (int i = threadIdx.x; i < kChunkTiles * kTkHistPad; i += kAgg) h[i] = 0;
    __syncthreads();
  }
  const int lane = lane_id();
  const int nw = (c.count + 63) >> 6;
  const int64_t W = lay.d_pad >> 6;
  const int64_t gw = c.start >> 6;
  // e_srv (mode 1) or x (mode 0), and the mean, over the chunk's elements:
  // past the chunk a load returns 0 and a store is dropped, so the pass has
  // no per-element branch (a store in one would make the loop wait for every
  // store before the next pass)
  const uint32_t nbytes = (uint32_t)c.count * 4u;
  const Buf rd = buf_of((kMode == 1 ? es : x) + c.start, nbytes);
  const Buf ra = buf_of(kAvg ? avg + c.start : es, kAvg ? nbytes : 0u);
  // Wave w takes the chunk's tiles w, w + kBW, ... one at a time, U words per
  // pass in word order, so that a tile's passes, and its list, are one
  // wave's.
  constexpr int kBW = kAgg / kWave;
  const auto next_w0 = [](int w) {
    return (w + U) % kTileWords != 0 ? w + U : w + U + (kBW - 1) * kTileWords;
  };
  bool bad = false;
  uint32_t lc = 0;  // list entries of the wave's tile so far
  // (past the chunk's last word, agg_words issues a load at a word that
  // exists and returns empty words: no branch, so no early wait)
  AggStep cur = agg_words<U>(sel, rank, W, gw, K, nw, wave_id() * kTileWords, 0, lane);
  // wait for the first words here, once: the loop header then knows them
  // loaded on both of its entries and does not wait at every pass for the
  // stores of the one before
  asm volatile("" ::"v"(cur.s), "v"(cur.r));
  for (int w0 = wave_id() * kTileWords; w0 < nw; w0 = next_w0(w0)) {
    float dv[U];
#pragma unroll
    for (int i = 0; i < U; ++i) dv[i] = buf_ld(rd, (uint32_t)((w0 + i) * 64 + lane) * 4u);
    float mean[U];
    if (kPath == kTkAggUnion) {
      // one batch holds every worker: the next pass's words go out first
      const AggStep nxt = agg_words<U>(sel, rank, W, gw, K, nw, next_w0(w0), 0, lane);
      const int wv = wave_id();
      union_means<U>(cur.words(), K, inv_k, vals + voff, tk.total_keep, keep, lane,
                     mb + wv * (U * kWave), wt + wv * kWave, ut + wv * U, mean);
      cur = nxt;
    } else {
      double acc[U];
#pragma unroll
      for (int i = 0; i < U; ++i) acc[i] = 0.0;
      for (int k0 = 0; k0 < K; k0 += kB) {
        // the next step's words go out before this step's values are waited for
        const bool last_b = k0 + kB >= K;
        const int nw0 = last_b ? next_w0(w0) : w0;
        const AggStep nxt =
            agg_words<U>(sel, rank, W, gw, K, nw, nw0, last_b ? 0 : k0 + kB, lane);
        const AggWords cw = cur.words();
        // This step's values, read through a buffer resource over each worker's
        // k_l values (a read past the end gets 0 from the range check, with no
        // memory access).
        bool done = false;
        if (kPath == kTkAggDense) {
          // Dense messages: the kept values of a worker's U words are contiguous
          // in its message; when no worker of the step has more than 64 of them,
          // one load per worker brings them all (lane j: the group's j-th
          // value) and each element takes its own with ds_bpermute.
          uint32_t gcnt = (uint32_t)(__popc(cw.lo) + __popc(cw.hi));
#pragma unroll
          for (int off = 1; off < U; off <<= 1) gcnt += (uint32_t)__shfl_xor((int)gcnt, off);
          if (__ballot(gcnt > (uint32_t)kWave) == 0ull) {  // wave-uniform
            float gv[kB];
#pragma unroll
            for (int kk = 0; kk < kB; ++kk) {
              const int kidx = min(k0 + kk, K - 1);  // absent workers have empty words
              const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                  (void*)(vals + (int64_t)kidx * tk.total_keep + voff), 0, (int)(keep * 4u),
                  kBufWord3);
              const uint32_t g4 = __builtin_amdgcn_readlane(cw.rk4, kk * U);  // group's first rank
              gv[kk] = __uint_as_float(
                  __builtin_amdgcn_raw_buffer_load_b32(rs, g4 + 4u * (uint32_t)lane, 0, 0));
            }
#pragma unroll
            for (int kk = 0; kk < kB; ++kk) {
              const uint32_t g4 = __builtin_amdgcn_readlane(cw.rk4, kk * U);
              // the U shuffles of the worker go out together (distinct
              // registers), then their values are added
              int pv[U];
#pragma unroll
              for (int i = 0; i < U; ++i) {
                const int q = kk * U + i;
                const uint32_t mlo = __builtin_amdgcn_readlane(cw.lo, q);
                const uint32_t mhi = __builtin_amdgcn_readlane(cw.hi, q);
                const uint32_t r4 = __builtin_amdgcn_readlane(cw.rk4, q);
                // the lane's element: its position among the group's kept values
                const uint32_t below =
                    __builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0u));
                const int src = (int)((r4 - g4) + 4u * below);  // < 4 * 64 for a kept element
                pv[i] = __builtin_amdgcn_ds_bpermute(src, __float_as_int(gv[kk]));
              }
#pragma unroll
              for (int i = 0; i < U; ++i) {
                const int q = kk * U + i;
                const uint32_t mlo = __builtin_amdgcn_readlane(cw.lo, q);
                const uint32_t mhi = __builtin_amdgcn_readlane(cw.hi, q);
                acc[i] += (double)sel_by_bit(((u64)mhi << 32) | mlo, __int_as_float(pv[i]),
                                             0.0f);  // worker order
              }
            }
            done = true;
          }
        }
        if (!done) {
          // Sparse messages (or a worker with more than 64 kept values in the
          // step's words): every (worker, word) pair gathers its values, a lane
          // whose bit is clear reading past the end; the loads go out before the
          // first one is used (dense kernels: one worker at a time, which needs fewer
          // registers next to the dense path).
          constexpr int kW = kPath == kTkAggDense ? 1 : kB;  // workers whose loads go out together
          for (int kw = 0; kw < kB; kw += kW) {
            float cv[kW][U];
#pragma unroll
            for (int kx = 0; kx < kW; ++kx) {
              const int kk = kw + kx;
              const int kidx = min(k0 + kk, K - 1);  // absent workers have empty words
              const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                  (void*)(vals + (int64_t)kidx * tk.total_keep + voff), 0, (int)(keep * 4u),
                  kBufWord3);
#pragma unroll
              for (int i = 0; i < U; ++i) {
                const int q = kk * U + i;
                const uint32_t mlo = __builtin_amdgcn_readlane(cw.lo, q);
                const uint32_t mhi = __builtin_amdgcn_readlane(cw.hi, q);
                const uint32_t r4 = __builtin_amdgcn_readlane(cw.rk4, q);
                // rank of the lane's element among the word's kept ones, in bytes
                const uint32_t below =
                    __builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0u));
                const uint32_t off =
                    sel_by_bit(((u64)mhi << 32) | mlo, below * 4u + r4, 0x80000000u);
                cv[kx][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
              }
            }
#pragma unroll
            for (int kx = 0; kx < kW; ++kx)
#pragma unroll
              for (int i = 0; i < U; ++i) acc[i] += (double)cv[kx][i];  // worker order; absent: +0
          }
        }
        cur = nxt;
      }
#pragma unroll
      for (int i = 0; i < U; ++i) mean[i] = (float)mean_of(acc[i], inv_k, K);
    }
    // the tile's list (kTkSpecCap entries; a store past it is dropped)
    const int tl = w0 / kTileWords;  // tile of the chunk
    const Buf rl = buf_of(tk.spec + ((int64_t)lay.k_max * lay.n_tiles + tile0 + tl) * kTkSpecCap,
                          kMode == 1 ? (uint32_t)kTkSpecCap * 8u : 0u);
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int j = (w0 + i) * 64 + lane;
      const bool ok = j < c.count;
      const uint32_t off = (uint32_t)j * 4u;
      if (kAvg) buf_st(ra, off, mean[i]);
      if (kMode == 1) {
        const float D = dv[i] + mean[i];  // Delta_{t+1} = e_t + (1/K) sum_k C(Delta^(k))
        buf_st(rd, off, D);
        const uint32_t key = key_of(D);
        bad |= ok && key >= kFiniteLimit;
        // list entry: Delta's bits | index in the tile << 32
        const u64 lm = __ballot(ok && key >= lo_spec);
        const uint32_t pos = lc + __builtin_amdgcn_mbcnt_hi((uint32_t)(lm >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)lm, 0u));
        u32x2 ev;
        ev.x = __float_as_uint(D);
        ev.y = (uint32_t)(j - tl * kTkTileElems);
        __builtin_amdgcn_raw_buffer_store_b64(
            ev, rl, ((lm >> lane) & 1ull) && pos < (uint32_t)kTkSpecCap ? pos * 8u : 0x80000000u,
            0, 0);
        lc += (uint32_t)__popcll(lm);
        // a pass stays in one tile; a lane past the chunk adds nothing
        const uint32_t hb = (uint32_t)(w0 / kTileWords) * kTkHistPad + hist_bin(key, win);
        // (the dense gathers lost with the leader: Top-5% 1.122-1.125 against
        // 1.111 ms, Top-10% 1.257 against 1.247-1.249 ms)
        if (kPath == kTkAggUnion)
          hist_add(h, hb, ok);
        else
          atomicAdd(&h[hb], ok ? 1u : 0u);
      } else {
        buf_st(rd, off, dv[i] - mean[i]);  // single-way: the mean itself comes back
      }
    }
    if (kMode == 1 && ((w0 + U) % kTileWords == 0 || w0 + U >= nw)) {
      // the tile's last pass: its list count (none before the first
      // threshold, for a tensor without lists, or past kTkSpecCap entries)
      if (lane == 0)
        tk.lcnt[(int64_t)lay.k_max * lay.n_tiles + tile0 + tl] =
            lo_spec != 0x80000000u && lc <= (uint32_t)kTkSpecCap ? lc : kTkSpecNone;
      lc = 0;
    }
  }
  if (kMode == 1) {
    if (__ballot(bad) != 0 && lane_id() == 0) atomicOr(lay.status, kStatusRange);
    __syncthreads();
    // the tile histograms of the chunk, 16-bit counts, two bins per store
    const int ntile = (c.count + kTkTileElems - 1) / kTkTileElems;
    uint32_t* out = reinterpret_cast<uint32_t*>(tile_hist(tk, lay, lay.k_max, tile0));
    for (int i = threadIdx.x; i < ntile * (kTkHistPad / 2); i += kAgg)
      out[i] = (h[2 * i] & 0xFFFFu) | (h[2 * i + 1] << 16);
  }
}

// ------------------------------------------------------------------ host side
struct Launcher {
  const DevLayout& lay;
  const TkDev& tk;
  hipStream_t s;

  // The Delta pass of R rows (row0..) over the part's tiles, with the step
  // ahead when st.xh is given; `start` stamps the dispatch's start when
  // non-null.
  hipError_t delta(const TkPart& p, int R, int row0, float lr, float mu, const float* g,
                   float* m, float* e, const uint64_t* psel, bool pend_in, const TkStep& st,
                   hipEvent_t start) const {
    const dim3 grid((unsigned)(run_padded_tiles(p.t1 - p.t0) * R));
#define SAEF_TKD(MOM, PEND, XH)                                                               \
  hipExtLaunchKernelGGL((k_tk_delta<MOM, PEND, XH>), grid, dim3(kBlock), kTkDeltaLdsPad, s,   \
                        start, nullptr, 0, lay, tk, p, R, row0, lr, mu, g, m, e, psel, st.x,  \
                        st.xh)
#define SAEF_TKD_X(MOM, PEND)                                                         \
  do {                                                                                \
    if (st.xh != nullptr) SAEF_TKD(MOM, PEND, true); else SAEF_TKD(MOM, PEND, false); \
  } while (0)
    if (m != nullptr) {
      if (pend_in) SAEF_TKD_X(true, true); else SAEF_TKD_X(true, false);
    } else {
      if (pend_in) SAEF_TKD_X(false, true); else SAEF_TKD_X(false, false);
    }
#undef SAEF_TKD_X
#undef SAEF_TKD
    return hipGetLastError();
  }

  // everything after the first pass for R rows of `data` (rows row0..) over
  // the part's tensors: the selection (pick; for a part with large tensors
  // the sums before it and gather and select, for the (row, tensor)s that the
  // pick left to them, after it), then the emit.  The last kernel stamps the
  // caller's stop event.
  hipError_t select_and_emit(const TkPart& p, int R, int row0, float* data, uint64_t* sel,
                             uint32_t* rank, float* vals, float* x, bool pend_out,
                             const LaunchEvents& last) const {
    const LaunchEvents ev;
    hipError_t err;
    const bool large = p.g1 > p.g0;
    const dim3 groups((unsigned)((int64_t)R * (p.g1 - p.g0)));
    const dim3 quarters((unsigned)((int64_t)R * (p.g1 - p.g0) * kGatherSplit));
    const dim3 pairs((unsigned)((int64_t)R * (p.l1 - p.l0)));
    const dim3 tiles((unsigned)((int64_t)(p.t1 - p.t0 + kWaves - 1) / kWaves * R));
    if (large) {
      SAEF_LAUNCH(k_tk_sum<false>, groups, dim3(kBlock), 0, s, lay, tk, p, row0);
      if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    if (p.s1 > p.s0) {
      SAEF_LAUNCH(k_tk_sum<true>, dim3((unsigned)((int64_t)R * (p.s1 - p.s0))), dim3(kBlock), 0,
                  s, lay, tk, p, row0);
      if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    if (tk.pick_wide != 0 || (tk.alone != 0 && pairs.x <= (unsigned)kTkWidePairs))
      SAEF_LAUNCH(k_tk_pick<kPickWide>, pairs, dim3(kPickWide), 0, s, lay, tk, p, row0, data);
    else
      SAEF_LAUNCH(k_tk_pick<kPick>, pairs, dim3(kPick), 0, s, lay, tk, p, row0, data);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    if (large) {
      if (tk.levels != 0) {
        SAEF_LAUNCH(k_tk_refine<0>, quarters, dim3(kBlock), 0, s, lay, tk, p, row0, data);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        SAEF_LAUNCH(k_tk_refine<1>, quarters, dim3(kBlock), 0, s, lay, tk, p, row0, data);
        if ((err = hipGetLastError()) != hipSuccess) return err;
      }
      // Up to 1.7 times the kept elements are listed: a chunk of 64 entries
      // holds the list of a tile of a sparse plan (up to 1/64 kept), else two
      // chunks of each tile are in flight together (Top-10%: 1064 us per
      // iteration with two, 1067 with four, 1101 against 1093 with one).
      // Up to a workgroup per CU, in a plan that is never split: a wave per tile
      // (with three times as many, 8.5 against 5.4 us: ragged tensors of 5 M
      // elements, K = 3).
      const bool sparse = tk.total_keep * 64 <= lay.d_pad;
      const bool wide = tk.alone != 0 && quarters.x <= (unsigned)kTkWidePairs;
      if (wide) {
        if (sparse)
          SAEF_LAUNCH((k_tk_gather<1, kGatherWide>), quarters, dim3(kGatherWide), 0, s, lay, tk, p,
                      row0, data);
        else
          SAEF_LAUNCH((k_tk_gather<2, kGatherWide>), quarters, dim3(kGatherWide), 0, s, lay, tk, p,
                      row0, data);
      } else if (sparse) {
        SAEF_LAUNCH((k_tk_gather<1, kBlock>), quarters, dim3(kBlock), 0, s, lay, tk, p, row0, data);
      } else {
        SAEF_LAUNCH((k_tk_gather<2, kBlock>), quarters, dim3(kBlock), 0, s, lay, tk, p, row0, data);
      }
      if ((err = hipGetLastError()) != hipSuccess) return err;
      // the select, with a workgroup per group (wide: per gather workgroup) that
      // mostly returns at once
      const dim3 picks((unsigned)((int64_t)R * (p.b1 - p.b0)) + (wide ? quarters.x : groups.x));
      if (wide)
        SAEF_LAUNCH(k_tk_select<kGatherSplit>, picks, dim3(kSelect), 0, s, lay, tk, p, R, row0,
                    data);
      else
        SAEF_LAUNCH(k_tk_select<1>, picks, dim3(kSelect), 0, s, lay, tk, p, R, row0, data);
      if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    if (x != nullptr)
      hipExtLaunchKernelGGL((k_tk_emit<true, false>), tiles, dim3(kBlock), 0, s, nullptr,
                            last.stop, 0, lay, tk, p, R, row0, data, sel, rank, vals, x);
    else if (pend_out)
      hipExtLaunchKernelGGL((k_tk_emit<false, true>), tiles, dim3(kBlock), 0, s, nullptr,
                            last.stop, 0, lay, tk, p, R, row0, data, sel, rank, vals, x);
    else
      hipExtLaunchKernelGGL((k_tk_emit<false, false>), tiles, dim3(kBlock), 0, s, nullptr,
                            last.stop, 0, lay, tk, p, R, row0, data, sel, rank, vals, x);
    return hipGetLastError();
  }

  // The server step over the part's tensors: the aggregation of the K
  // messages, then (mode 1) the server row's selection and message.  The
  // aggregation stamps ev.start; the last kernel ev.stop.
  hipError_t server(const TkPart& p, int K, int mode, const uint64_t* sel, const uint32_t* rank,
                    const float* vals, float* avg, float* e_srv, uint64_t* srv_sel,
                    uint32_t* srv_rank, float* srv_vals, float* x,
                    const LaunchEvents& ev) const {
    const dim3 grid((unsigned)(p.c1 - p.c0));
    const double ik = inv_pow2(K);
    hipEvent_t stop0 = mode == 1 ? nullptr : ev.stop;
    // dense messages (at least 1/32 of the elements kept): one load per worker
    // and step, values handed out with ds_bpermute; sparser ones: gathers over
    // the union of the workers' kept elements when one batch holds every
    // worker (K <= 16), else per-pair gathers.  At resnet50 K = 8 the union
    // took the Top-1% iteration from 1.000 to 0.984 ms (its end, pipelined:
    // 710 -> 680 us); for dense messages it lost to the one-load-per-worker
    // path (Top-5% 1.12 against 1.11 ms, Top-10% 1.29 against 1.25 ms).
    const bool co = tk.total_keep * 32 >= lay.d_pad;
#define SAEF_TKA(M, A, U, C)                                                                 \
  hipExtLaunchKernelGGL((k_tk_aggregate<M, A, U, C>), grid, dim3(kAgg), 0, s, ev.start, stop0, \
                        0, lay, tk, p, K, ik, sel, rank, vals, avg, e_srv, x)
#define SAEF_TKA_U(M, A)                                                    \
  do {                                                                      \
    if (K <= 8) {                                                           \
      if (co) SAEF_TKA(M, A, 8, kTkAggDense);                               \
      else SAEF_TKA(M, A, 8, kTkAggUnion);                                  \
    } else if (K <= 16) {                                                   \
      if (co) SAEF_TKA(M, A, 4, kTkAggDense);                               \
      else SAEF_TKA(M, A, 4, kTkAggUnion);                                  \
    } else {                                                                \
      if (co) SAEF_TKA(M, A, 4, kTkAggDense);                               \
      else SAEF_TKA(M, A, 4, kTkAggPairs);                                  \
    }                                                                       \
  } while (0)
    if (mode == 1) {
      if (avg != nullptr) SAEF_TKA_U(1, true); else SAEF_TKA_U(1, false);
    } else {
      if (avg != nullptr) SAEF_TKA_U(0, true); else SAEF_TKA_U(0, false);
    }
#undef SAEF_TKA_U
#undef SAEF_TKA
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess || mode != 1) return err;
    return select_and_emit(p, 1, lay.k_max, e_srv, srv_sel, srv_rank, srv_vals, x, false, ev);
  }
};

}  // namespace

// After a fork, an error still joins: s waits for whatever the side stream
// was given, so no work of this call outlives it on the side stream.
static hipError_t join_side(hipStream_t s, const TkStreams& side, hipError_t err) {
  const hipError_t e1 = hipEventRecord(side.join, side.stream);
  const hipError_t e2 = e1 == hipSuccess ? hipStreamWaitEvent(s, side.join, 0) : e1;
  return err != hipSuccess ? err : e2;
}

hipError_t launch_topk_compress(const DevLayout& lay, const TkDev& tk, const TkPart& all, int K,
                                float lr, float mu, const float* g, float* m, float* e,
                                uint64_t* sel, uint32_t* rank, float* vals, bool pend_in,
                                bool pend_out, const TkStep& st, hipStream_t s,
                                const TkStreams& side, const LaunchEvents& ev) {
  // The Delta pass of a group of rows is HBM-bound; the selection chain that
  // follows it (sums, pick, gather, select, emit) is mostly launch- and
  // latency-bound.  With a side stream the workers are taken in two groups: the first group's chain runs on the side stream while the
  // second group's Delta pass streams on s; s waits for the side stream at
  // the end.  The groups' scratch rows are disjoint.
  const bool split = side.stream != nullptr && K >= 2;
  const int R0 = split ? (K + 1) / 2 : K;
  const Launcher main{lay, tk, s};
  const int64_t W = lay.d_pad >> 6;
  // the first Delta pass stamps the start event, the last kernel on s the stop event
  hipError_t err = main.delta(all, R0, 0, lr, mu, g, m, e, sel, pend_in, st, ev.start);
  if (err != hipSuccess) return err;
  if (!split) return main.select_and_emit(all, K, 0, e, sel, rank, vals, nullptr, pend_out, ev);
  const int R1 = K - R0;
  if ((err = hipEventRecord(side.fork, s)) != hipSuccess) return err;
  if ((err = hipStreamWaitEvent(side.stream, side.fork, 0)) != hipSuccess) return err;
  const Launcher aside{lay, tk, side.stream};
  err = aside.select_and_emit(all, R0, 0, e, sel, rank, vals, nullptr, pend_out, LaunchEvents());
  if (err == hipSuccess) err = main.delta(all, R1, R0, lr, mu, g, m, e, sel, pend_in, st, nullptr);
  if (err == hipSuccess)
    err = main.select_and_emit(all, R1, R0, e + (int64_t)R0 * lay.d_pad, sel + (int64_t)R0 * W,
                               rank + (int64_t)R0 * W, vals + (int64_t)R0 * tk.total_keep,
                               nullptr, pend_out, ev);
  return join_side(s, side, err);
}

hipError_t launch_topk_round_end(const DevLayout& lay, const TkDev& tk, const TkPart* parts,
                                 int n_parts, int K, float lr, float mu, int mode,
                                 const float* g, float* m, float* e, uint64_t* sel,
                                 uint32_t* rank, float* vals, bool pend_in, float* e_srv,
                                 uint64_t* srv_sel, uint32_t* srv_rank, float* srv_vals,
                                 float* x, const TkStep& st, hipStream_t s,
                                 const TkStreams& side, const LaunchEvents& ev) {
  // Every step after the Delta pass works tensor by tensor, so the parts are
  // independent once their Delta is formed: the Delta passes of the parts
  // stream one after another on s, and each part but the last, as soon as
  // its Delta is stored, runs its worker selection and messages and its
  // server step on the side stream, under the next parts' Delta passes; the
  // last part's steps run on s, which then waits for the side stream.  All
  // data and scratch of two parts are disjoint (tiles, groups, chunks and
  // (row, tensor) state).
  const Launcher main{lay, tk, s};
  const Launcher aside{lay, tk, side.stream};
  hipError_t err = hipSuccess;
  bool forked = false;
  for (int i = 0; i < n_parts && err == hipSuccess; ++i) {
    const TkPart& p = parts[i];
    const bool last = i == n_parts - 1;
    err = main.delta(p, K, 0, lr, mu, g, m, e, sel, pend_in, st, i == 0 ? ev.start : nullptr);
    if (err == hipSuccess && !last) {
      err = hipEventRecord(side.fork, s);
      if (err == hipSuccess) err = hipStreamWaitEvent(side.stream, side.fork, 0);
      forked = forked || err == hipSuccess;
    }
    const Launcher& on = last ? main : aside;
    if (err == hipSuccess)
      err = on.select_and_emit(p, K, 0, e, sel, rank, vals, nullptr, true, LaunchEvents());
    LaunchEvents tail;
    if (last) tail.stop = ev.stop;
    if (err == hipSuccess)
      err = on.server(p, K, mode, sel, rank, vals, nullptr, e_srv, srv_sel, srv_rank, srv_vals,
                      x, tail);
  }
  return forked ? join_side(s, side, err) : err;
}

// Grid: n_tiles * K workgroups; workgroup b sets to 0 the elements of worker
// b % K's tile b / K whose selection bit is set (wave w: words w*kTkU ..).
__global__ __launch_bounds__(kBlock) void k_tk_zero(DevLayout lay, int K, float* __restrict__ e,
                                                    const uint64_t* __restrict__ sel) {
  const int k = (int)(blockIdx.x % (unsigned)K);
  const int64_t ti = blockIdx.x / (unsigned)K;
  const Tile tile = lay.tiles[ti];
  const int nw = (tile.count + 63) >> 6;
  const int lane = lane_id();
  const uint64_t* sk = sel + (int64_t)k * (lay.d_pad >> 6) + (tile.start >> 6);
  float* ek = e + (int64_t)k * lay.d_pad + tile.start;
  for (int w = wave_id() * kTkU; w < min(nw, wave_id() * kTkU + kTkU); ++w) {
    const u64 word = sk[w];
    const int j = w * 64 + lane;
    if (((word >> lane) & 1ull) && j < tile.count) ek[j] = 0.0f;
  }
}

hipError_t launch_topk_materialize(const DevLayout& lay, int K, float* e, const uint64_t* sel,
                                   hipStream_t s, const LaunchEvents& ev) {
  const dim3 grid((unsigned)(lay.n_tiles * K));
  SAEF_LAUNCH(k_tk_zero, grid, dim3(kBlock), 0, s, lay, K, e, sel);
  return hipGetLastError();
}

hipError_t launch_topk_aggregate(const DevLayout& lay, const TkDev& tk, const TkPart& all,
                                 int K, int mode, const uint64_t* sel, const uint32_t* rank,
                                 const float* vals, float* avg, float* e_srv, uint64_t* srv_sel,
                                 uint32_t* srv_rank, float* srv_vals, float* x, hipStream_t s,
                                 const LaunchEvents& ev) {
  return Launcher{lay, tk, s}.server(all, K, mode, sel, rank, vals, avg, e_srv, srv_sel,
                                     srv_rank, srv_vals, x, ev);
}

}  // namespace saef
