// Internal declarations of the layer-wise Top-K compressor (kernels in
// saef_topk.hip, entry points in saef_api.hip); not part of the public C ABI.
#pragma once

#include "saef_internal.h"

namespace saef {

// Pass-1 histogram of the key |v| around the threshold tau of the previous
// call: a near range of kTkNear bins of 1/512 binade from kTkSpecMargin (1/32
// binade) under tau to 0.19 binades above it; below it kTkMidB bins of 1/64
// binade (to 1.16 binades under tau), then kTkFarB of 1/8 (to 3.66); above it
// kTkMidA bins of 1/64 (to 0.81 binades over tau), then kTkFarA of 1/8 (to
// 2.06); on each side one open bin.  The bins only decide how many elements
// become candidates; the kept set is exact wherever the threshold falls.  Under
// error feedback the residual piles up at tau; tau rises by 0.01-0.2 binades a
// call (resnet50) and falls by 0.5-1.1 when the errors are averaged (up to 2
// for 16 independent ones).  A bin of 1/64 binade at tau held 5000-7000 of the
// 2.36 M elements of the largest tensors at Top-1% and 17000-29000 at Top-10%,
// and selecting among them was most of the selection's time; 160 bins of
// 1/2048 binade, or 224 of 1/512 with coarse ones below, miss the moves
// (Top-10% 1195 and 1154 against 1110 us).
constexpr int kTkSubShift = 14;                // near bin width: 2^14 keys
constexpr int kTkNear = 112;                   // near bins
constexpr int kTkMidShift = 17;                // mid bin width: 2^17 keys
constexpr int kTkMidB = 72;                    // below: 1.125 binades
constexpr int kTkMidA = 40;                    // above: 0.625 binades
constexpr int kTkFarShift = 20;                // far bin width: 2^20 keys
constexpr int kTkFarB = 20;                    // 2.5 binades
constexpr int kTkFarA = 10;                    // 1.25 binades
constexpr int kTkBelow = kTkMidB + kTkFarB + 1;  // bins below the near range
constexpr int kTkAbove = kTkMidA + kTkFarA + 1;  // bins above it
constexpr int kTkHist = kTkBelow + kTkNear + kTkAbove;
constexpr int kTkHistPad = 256;                // 16-bit counts per tile
constexpr int kTkGroup = 64;      // tile histograms (or group sums) one sum workgroup adds
constexpr int kTkSmall = 16;      // most tiles of a small tensor in a plan with more than a group
// The pick has 1024 threads where some small tensor has more than kTkPickTiles
// tiles (a wave takes them one after another), and in a plan that is never
// split where at most kTkWidePairs (row, tensor)s are picked, a workgroup for
// each CU: 30 tensors of 18 tiles, K = 8, Top-20% 134 us per iteration against
// 157 with 256 threads, one of 16 tiles, K = 2, 75.5 against 96.4, one of 32
// 90 against 131.  With more pairs their waves are in each other's way
// (resnet56, 1336 pairs: 128 against 97 us), and beside a Delta pass they wait
// for slots (resnet50 Top-1%: 851 against 819).
constexpr int kTkPickTiles = 20;
constexpr int kTkWidePairs = 256;
// Fewest (tile, worker) pairs of a call that is split over the side stream: a
// smaller one streams its Delta in a few microseconds, and a second chain of
// kernels costs more than it hides (resnet56 K = 8, 4160 pairs: 120 us per
// Top-5% iteration whole, 131 split; ragged K = 3, 7400 pairs: 262 against
// 284 us; resnet50 K = 8 has 100,000).
constexpr int64_t kTkSplitTiles = 16384;
constexpr int kTkRefineLevels = 2;  // histograms of 11 key bits a refined bin gets
// Gather workgroups per group of tiles (a wave then takes 4 tiles; 8 groups of
// 2: resnet50 Top-1% 872 against 850 us, bert_base 7.48 against 7.13 ms; 16 of
// one: 929 us and 8.69 ms).
constexpr int kTkGatherSplit = 4;
constexpr int kTkBins = 2048;     // bins of an 11-bit radix digit
// Elements per server-aggregation workgroup: four tiles, one per wave.  Its 17
// KB of LDS let it run beside a Delta pass, and a small layout still fills
// the chip (resnet56 Top-5%: 120 us per iteration, 123 at 8 tiles, 136 at 16;
// with 32 tiles in 1024 threads the kernel took 39 us there against 19).
constexpr int kTkChunk = 8192;
// Speculative candidate lists: for a tensor that keeps at most 1/8 of its
// elements, the worker Delta pass also writes, per (row, tile), the elements
// whose key is at least the previous call's threshold key minus
// kTkSpecMargin (1/32 binade), in index order, up to kTkSpecCap of them, and
// their count (kTkSpecNone when the tile had more); the server aggregation
// does the same for the server row.  When the bin b1 that this call's
// histogram picks lies at or above that bound, the list holds every element
// the selection needs and the tile's Delta is not read again; otherwise the
// selection reads Delta and writes the list again down to that bin, for the emit.
// (Under error feedback the threshold mostly rises from call to call, and the
// elements just below it pile up: at 1% kept the lists hold about 3% of the
// elements.)
constexpr int kTkSpecCap = 512;
constexpr uint32_t kTkSpecNone = 0xFFFFu;
constexpr uint32_t kTkSpecMargin = 1u << 18;
static_assert(kTkMidB % (1 << (kTkFarShift - kTkMidShift)) == 0 &&
                  kTkMidA % (1 << (kTkFarShift - kTkMidShift)) == 0,
              "the mid bins of a side are whole far bins");
constexpr int kTkSpecMaxShare = 8;  // lists when k_l * 8 <= n_l
// Dynamic LDS the Delta pass requests and does not use: with its own 1 KB
// it keeps at most 5 of its workgroups on a CU (160 KB of LDS), so the
// selection kernels of the other rows or tensors, launched on the side
// stream while a Delta pass streams, find free slots.  At resnet50 K = 8
// Top-1% per iteration: 1.014 ms against 1.030 ms uncapped, 1.017 ms with
// only the overlapped pass capped, 1.022 ms at 4 workgroups per CU.  With the
// step ahead in the pass: 0.876 ms at 5, 0.879 at 4, 0.887 at 6, 0.929 at 3.
constexpr unsigned kTkDeltaLdsPad = 26624;
// The Top-K kernels take a tile as 32 sign words (one per lane of a gather
// wave): they need the layout's tiles to hold 2048 elements.  A library built
// with another SAEF_TILE_ELEMS (the sign path works with any) refuses Top-K
// plans (saef_topk_create returns SAEF_EINVAL).
constexpr int kTkTileElems = 2048;
constexpr bool kTkUsable = kTileElems == kTkTileElems;
static_assert(kTkHistPad >= kTkHist && kTkHistPad % 4 == 0, "padded tile histogram");
static_assert(kTkTileElems < 65536, "a tile's bin counts fit 16 bits");
static_assert(kTkChunk % kTkTileElems == 0, "a server chunk holds whole tiles");
static_assert(kTkSpecCap < (int)kTkSpecNone, "list counts fit the slot below the marker");
static_assert((int64_t)kTileElems * kMaxTilesPerTensor >= kMaxTensor,
              "every tensor is cut into tiles of kTileElems elements");

// Up to kTkChunk elements of one tensor (whole tiles): the server's workgroups.
struct TkChunk {
  int64_t start;  // absolute element index (multiple of 64)
  int32_t l;
  int32_t count;
};

// kTkGroup consecutive tiles of one tensor (a group), or kTkGroup consecutive
// groups of one tensor (a super-group).
struct TkGroup {
  int32_t l;
  int32_t first;  // first tile (group) index, global
  int32_t n;      // tiles (groups) in it
  int32_t pad;
};

struct TkTensor {
  int64_t voff;         // first value of the tensor in a message
  int64_t keep;         // k_l
  int32_t first_chunk;  // server chunks
  int32_t nchunks;
  int32_t first_group;  // tile groups, for a large tensor (more than kTkGroup tiles; more than
                        // kTkSmall in a plan that has one of more than kTkGroup)
  int32_t ngroups;      // 0 otherwise
  int32_t first_sgroup;  // super-groups, when ngroups > kTkGroup (a huge tensor)
  int32_t nsgroups;      // 0 otherwise
  int32_t large;         // number among the large tensors
  int32_t pad;
};

// Selection state of one (row, tensor).  Kept from one call to the next:
// the threshold key tau, the last kept index iota (in the tensor) of the
// elements equal to tau, and the histogram's near range placed at tau.  Set by
// the pick: the lists' bound of this call, and for a large tensor the key
// range [lo, up) of the candidates (the bin that holds the k-th largest key),
// how many of them to take, and whether there are many of them.
struct TkSel {
  uint32_t tau;
  uint32_t win;     // first key of the histogram's near range
  uint32_t floor;   // the lists hold every element with a key >= floor (2^31: no lists); once the
                    // gather has been over them, at most its lo
  uint32_t lists;   // 1: the rows of this tensor keep speculative lists (set at creation)
  uint32_t lo, up;
  uint32_t coarse;  // 1: [lo, up) is full: its keys are counted into rhist
  uint32_t pad;
  int64_t need;
  int64_t iota;     // elements equal to tau with index <= iota are kept
};

// A run of whole tensors [l0, l1) with the tiles, tile groups, super-groups
// and server chunks that belong to them: each a contiguous index range, since
// all four are numbered tensor by tensor.  The Top-K kernels work on one
// part; the whole layout is one part.
struct TkPart {
  int32_t l0, l1;  // tensors
  int32_t t0, t1;  // tiles
  int32_t g0, g1;  // tile groups
  int32_t s0, s1;  // super-groups
  int32_t c0, c1;  // server chunks
  int32_t b0, b1;  // large tensors
};

struct TkDev {
  const TkChunk* chunks;
  const TkTensor* tens;
  const TkGroup* groups;
  const TkGroup* sgroups;
  uint16_t* thist;     // [rows][n_tiles][kTkHistPad] tile histograms
  uint32_t* ghist;     // [rows][n_groups][kTkHistPad] group sums
  uint32_t* sghist;    // [rows][n_sgroups][kTkHistPad] super-group sums
  TkSel* sel;          // [rows][L]
  uint32_t* tile_cnt;  // [rows][n_tiles] kept per tile, then the exclusive prefix
  uint32_t* lcnt;      // [rows][n_tiles] entries in the tile's speculative list, or kTkSpecNone
  uint32_t* rhist;     // [rows][n_large][kTkRefineLevels][kTkBins] histograms of full bins
  uint32_t* tile_cand;  // [rows][n_tiles] candidates of the tile (full bins)
  uint32_t* seg;       // [rows][n_groups * kTkGatherSplit] candidates of each gather workgroup
  uint32_t* arrived;   // [rows][n_large] workgroups of the select that gathered; 0 between calls
  const int32_t* large;  // [n_large] the large tensors, in order
  // [rows][d_pad] candidate slots: (row, tensor) at the tensor's offset, those
  // of a gather workgroup at its first tile
  unsigned long long* cand;
  unsigned long long* spec;  // [rows][n_tiles][kTkSpecCap] Delta's bits | (index in the tile) << 32
  int64_t n_chunks;
  int64_t n_groups;
  int64_t n_sgroups;
  int64_t n_large;     // large tensors (those with tile groups)
  int64_t total_keep;
  int32_t levels;      // times the refine may narrow a full bin: kTkRefineLevels when some
                       // tensor has super-groups, else 0 (no refine: the gather counts and
                       // the select's launch gathers)
  int32_t pick_wide;   // 1: some small tensor has more than kTkPickTiles tiles
  int32_t alone;       // 1: no call of the plan is split over the side stream
  int32_t pad;
};

// Worker Top-K compression of K rows (row k of e, histogram row k).  m
// non-null: momentum.  Writes Delta into e, the selection words, rank words
// and values of each row.  pend_in: e holds the previous call's Delta whose
// kept elements (the selection words in sel) are still to be set to 0; they
// are read as 0.  pend_out: this call's kept elements are left as they are
// (pending, for the next reader) instead of being set to 0.
//
// side: a second stream of the plan and two events (fork, join).  When
// given and K >= 2, the rows are compressed in two groups and the first
// group's selection runs on the side stream, overlapping the second group's
// Delta pass; s waits for the side stream before the call returns (an event
// fork and join, so the launches stay capturable in a HIP graph).
struct TkStreams {
  hipStream_t stream = nullptr;
  hipEvent_t fork = nullptr;
  hipEvent_t join = nullptr;
};
// The iteration's step ahead xh = x - e taken along by the Delta pass (xh
// null: not).
struct TkStep {
  const float* x = nullptr;
  float* xh = nullptr;
};
// `all`: the part of every tensor.
hipError_t launch_topk_compress(const DevLayout& lay, const TkDev& tk, const TkPart& all, int K,
                                float lr, float mu, const float* g, float* m, float* e,
                                uint64_t* sel, uint32_t* rank, float* vals, bool pend_in,
                                bool pend_out, const TkStep& st, hipStream_t s,
                                const TkStreams& side,
                                const LaunchEvents& ev = LaunchEvents());

// Sets to 0 the elements of the K rows of e whose selection bit is set.
hipError_t launch_topk_materialize(const DevLayout& lay, int K, float* e, const uint64_t* sel,
                                   hipStream_t s, const LaunchEvents& ev = LaunchEvents());

// Server Top-K aggregation: mean of the K decoded messages; mode 1: e_srv
// <- e_srv + mean, its Top-K message, e_srv at kept elements <- 0 and x <- x
// - C(Delta); mode 0: x <- x - mean.  avg written when non-null.
hipError_t launch_topk_aggregate(const DevLayout& lay, const TkDev& tk, const TkPart& all,
                                 int K, int mode, const uint64_t* sel, const uint32_t* rank,
                                 const float* vals, float* avg, float* e_srv, uint64_t* srv_sel,
                                 uint32_t* srv_rank, float* srv_vals, float* x, hipStream_t s,
                                 const LaunchEvents& ev = LaunchEvents());

// The worker compression (pend_out: its kept elements left pending) and the
// server step of one iteration, pipelined over n_parts >= 2 parts that
// cover the tensors in order: the parts' Delta passes run one after another
// on s, and each part but the last then takes its selection, messages and
// server step on the side stream while the later parts' Delta passes
// stream; s waits for the side stream at the end (an event fork and join).
// The same results as launch_topk_compress then launch_topk_aggregate (avg
// null).  ev: start stamped by the first Delta pass, stop by the last kernel
// on s.
hipError_t launch_topk_round_end(const DevLayout& lay, const TkDev& tk, const TkPart* parts,
                                 int n_parts, int K, float lr, float mu, int mode,
                                 const float* g, float* m, float* e, uint64_t* sel,
                                 uint32_t* rank, float* vals, bool pend_in, float* e_srv,
                                 uint64_t* srv_sel, uint32_t* srv_rank, float* srv_vals,
                                 float* x, const TkStep& st, hipStream_t s,
                                 const TkStreams& side, const LaunchEvents& ev = LaunchEvents());

}  // namespace saef
