// Host-side geometry of the launches: how a layout is cut into chunks, which kernels a layer takes and
// how large their grids are. Plain C++ on integers, without HIP, so that it is checked on the host over
// all shapes.
#pragma once

#include <algorithm>
#include <limits.h>
#include <stddef.h>
#include <stdint.h>

#include "epl.h"

namespace epl {

constexpr int kWave = 64;
constexpr int kLayoutThreads = 256;
constexpr int kLayoutWaves = kLayoutThreads / kWave;
// Pairs handled by one layout workgroup ("chunk"); a chunk never spans two source ranks and
// always holds whole tokens.
constexpr int kMaxChunkPairs = 1024;

// Shape of one layout problem, derived on the host from epl_config.
struct Geom {
  int R, E, El, k, Tr;
  int CT;     // tokens per chunk
  int NC;     // chunks per source rank (>= 1)
  int nblk;   // R * NC layout workgroups
  int ebits;  // bits needed for an expert id (ballot-match key width)
  int rbits;  // bits needed for a rank id
  float inv_k, inv_El, inv_R;  // 1/k, 1/El, 1/R for exact small quotients
  int64_t T;
};

inline int bits_for(int n) {  // bits needed to represent values 0..n-1
  int b = 0;
  while ((1 << b) < n) ++b;
  return b;
}

// Chunking of each source rank's tokens for the layout kernels: whole tokens, at most
// kMaxChunkPairs pairs per workgroup.
inline Geom make_geom(int R, int E, int k, int Tr) {
  Geom g;
  g.R = R;
  g.E = E;
  g.El = g.E / g.R;
  g.k = k;
  g.Tr = Tr;
  g.T = (int64_t)g.R * g.Tr;
  // Aim for >= 256 workgroups (the chip has 256 CUs) and >= 64 pairs per workgroup, with at
  // most kMaxChunkPairs pairs per chunk.
  const int cap = kMaxChunkPairs / g.k;  // k <= 32 so cap >= 32
  const int64_t want = std::max<int64_t>((g.T + 255) / 256, (64 + g.k - 1) / g.k);
  const int ct = (int)std::min<int64_t>(want, cap);
  g.CT = g.Tr < 1 ? 1 : std::min(ct, g.Tr);
  g.NC = g.Tr < 1 ? 1 : (g.Tr + g.CT - 1) / g.CT;
  g.nblk = g.R * g.NC;
  g.ebits = bits_for(g.E);
  g.rbits = bits_for(g.R);
  g.inv_k = 1.0f / (float)g.k;
  g.inv_El = 1.0f / (float)g.El;
  g.inv_R = 1.0f / (float)g.R;
  return g;
}

// ------------------------------------------------------------------------ layouts in one launch
// The one-launch layout (small.hip) counts all T*k ids in every workgroup and deduplicates each source
// rank's earlier tokens again, so it is used only up to these sizes; larger layouts take three
// launches. Whole layer of 2048 columns, layout and dispatch in one launch against three: 16K pairs
// on 32 ranks 35.9 / 39.2 us, 24K 56.2 / 55.2, 32K 71.6 / 69.2. The rank limit keeps the second pass
// short: 16K pairs on one rank took 39.7 / 37.5 us, 16K of top-1 67.6 / 44.2, 12K on two ranks
// 29.2 / 32.1.
constexpr int64_t kSingleMaxPairs = 16384;     // T*k
constexpr int64_t kSingleMaxRankPairs = 4096;  // Tr*k
// Bound on 9 E + 6 R for epl_layout alone, whose launch count (epl_layout_launches) it is part of; the kernel
// needs none. epl_layout_dispatch and its phases have no such bound: 4K pairs on 1024 ranks of one expert take 26.6 us
// per layer in one launch, 51.9 with a three-launch layout.
constexpr int64_t kSingleMaxTable = 12287;

inline bool small_layout(const Geom& g) {
  return g.T * g.k <= kSingleMaxPairs && (int64_t)g.Tr * g.k <= kSingleMaxRankPairs;
}

inline bool layout_single(const Geom& g) {  // true if epl_layout runs as one launch for this geometry
  return small_layout(g) && 9 * (int64_t)g.E + 6 * g.R <= kSingleMaxTable;
}

// Tokens per group. Every group repeats the pass over all ids, so fewer groups are cheaper; but a
// group also sends its tokens' rows with four waves only, so more groups hide more latency.
// * Layout alone: 256 groups, one per compute unit, at most a wave of pairs each (layout of 16K
//   pairs and dispatch and combine of 2048-wide rows, us for 256 / 512 / 1024 / 2048 groups: 38.2 /
//   39.4 / 43.1 / 48.8).
// * With the send: one 4 KiB piece (an fp8 pass) per wave, as long as the groups' passes stay under
//   kSmallMaxCounts ids in all. Whole layer, us for 256 / 512 / 1024 / 2048 groups: 4.7K pairs of
//   5120 columns 49.3 / 46.6 / 45.2 / 41.9; 8K pairs of 7168 57.3 / 56.3 / 55.6 / 55.6; 16K of 7168
//   109.0 / 108.3 / 105.9 / 105.9; 16K of 2048 35.5 / 36.0 / 37.1 / 41.8; 16K (top-1) of 1024 44.2 /
//   41.3 / 42.9 / 50.5.
constexpr int64_t kSmallMaxCounts = 1 << 24;
inline int group_tokens(const Geom& g, int pieces) {
  const int64_t most = std::min<int64_t>(kWave / g.k, (g.T + 255) / 256);
  const int64_t want = pieces ? std::max<int64_t>(kLayoutWaves / pieces, (g.T * g.T * g.k + kSmallMaxCounts - 1) / kSmallMaxCounts)
                              : most;
  return (int)std::max<int64_t>(1, std::min(want, most));
}

// Whether epl_layout_dispatch takes one launch for the layout and its rows (small.hip), or the rows a second
// one. Every group of tokens counts all ids again and then sends with four waves, so many tokens are better
// sent by the row kernel. Layout, dispatch and combine, speed in one launch / in two against a layout whose
// workgroups walked each token's choices, followed by the row kernel; bf16 rows of 128 columns on 4 ranks:
// top-1 of 2816 tokens 1.21 / 1.15, 4096 1.04 / 1.14, 8192 0.74 / 1.05, 16384 0.78 / 1.00; top-4 of 2816 tokens
// 1.05 / 1.08, 4096 0.75 / 1.02; top-5 of 2816 1.01 / 1.07. T*T*k stands for the ids that all groups count.
// fp8 rows are quantised a 1024-column pass to a wave, at an occupancy that suits counting and not
// quantising: top-2 on 4 ranks, 1536 tokens of 3072 columns 1.10 / 1.09, 2048 tokens 0.96 / 1.09; top-6,
// 1536 x 3072 0.97 / 1.05; top-4, 2048 x 4096 0.93 / 1.02; top-8, 1536 x 7168 1.07 / 1.03.
constexpr int64_t kSmallSendTokens = 2816;
constexpr int64_t kSmallSendTokens1 = 4096;    // top-1, from four ranks on
constexpr int64_t kSmallSendCounts = 1 << 25;  // T*T*k
constexpr int64_t kSmallSendPasses = 4096, kSmallSendPassesMany = 3072;  // fp8, tokens * passes up to / beyond top-4
constexpr int64_t kSmallSendWide = 1536;       // fp8, rows of as many passes as a group has waves, or more: tokens
inline int small_pieces(int H, bool fp8) { return fp8 ? (H + 1023) / 1024 : (H + 2047) / 2048; }  // of a row: passes, or 4 KiB
inline bool small_dispatch(const Geom& g, int H, bool fp8) {
  if (!small_layout(g)) return false;
  const int pieces = small_pieces(H, fp8);
  // Ranks so short that the layout alone would take as many groups: sending with them costs no counting
  // (1024 ranks of 16 tokens, top-1 x 512 columns: 42.0 us in one launch, 45.8 in two).
  if (g.Tr <= group_tokens(g, pieces)) return true;
  if (g.T > (g.k == 1 && g.R >= 4 ? kSmallSendTokens1 : kSmallSendTokens) || g.T * g.T * g.k > kSmallSendCounts) return false;
  return !fp8 || g.T <= (pieces >= kLayoutWaves ? kSmallSendWide : (g.k <= 4 ? kSmallSendPasses : kSmallSendPassesMany) / pieces);
}

// ------------------------------------------------------------------------ layouts in two launches
// route_count and route_place (layout.hip), for layouts of few chunks.
constexpr int kPlaceMaxChunks = 512;
constexpr int kPlaceLanes = 32;    // threads that read one row of counts, 16 bytes (eight experts) each
constexpr int kPlaceRows = kLayoutThreads / kPlaceLanes;  // rows read side by side
constexpr int kPlaceExperts = 8 * kPlaceLanes;
constexpr int kPlaceAhead = 8;     // group rows in flight per thread
constexpr int kGroupChunks = 4;    // chunks whose counts route_count also sums

// The chunks that are launched. A few chunks past 256 (where the source ranks do not divide it) would
// make every workgroup wait for a second batch of group rows: 264 chunks took 8.1 us, 256 6.5. Slightly
// longer chunks avoid it, so there are never more of them than in g (the workspace is sized for g).
inline Geom place_geom(const Geom& geom) {
  Geom g = geom;
  constexpr int kOneBatch = kPlaceAhead * kPlaceRows * kGroupChunks;
  if (g.nblk > kOneBatch && g.R <= kOneBatch) {
    const int per_rank = kOneBatch / g.R;
    g.CT = std::min((g.Tr + per_rank - 1) / per_rank, kMaxChunkPairs / g.k);
    g.NC = (g.Tr + g.CT - 1) / g.CT;
    g.nblk = g.R * g.NC;
  }
  return g;
}

// Bound on the pairs of the group rows that one thread of route_place adds up. Every run of NC chunks
// holds one rank's tokens, so a group of kGroupChunks holds as many whole ranks' as fit, and at most CT
// tokens in each chunk that is left.
inline int64_t place_sum(const Geom& launched) {
  const Geom& g = launched;
  const int64_t rows = (g.nblk + kGroupChunks * kPlaceRows - 1) / (kGroupChunks * kPlaceRows);
  const int64_t tokens = (int64_t)(kGroupChunks / g.NC) * g.Tr + (int64_t)(kGroupChunks % g.NC) * g.CT;
  return rows * tokens * g.k;
}

// Layouts whose count matrix every workgroup of route_place can sum for itself, in 16-bit halves.
inline bool place_layout(const Geom& g) {
  return g.E <= kPlaceExperts && g.nblk <= kPlaceMaxChunks && place_sum(place_geom(g)) < 65536;
}

// Kernels that epl_layout_dispatch launches: the layout with its rows, or the layout's launches and the rows'.
inline int layout_dispatch_launches(const Geom& g, int H, bool fp8) {
  if (small_dispatch(g, H, fp8)) return 1;
  return small_layout(g) ? 2 : place_layout(g) ? 3 : 4;
}

// ------------------------------------------------------------------------ row kernels
// Workgroups for `units` units, `per_group` to a workgroup of `threads` threads, of a kernel that strides
// over its units. HIP takes fewer than 2^32 threads per grid dimension (gridDim * blockDim), which 1 KiB
// units of a 64 GiB x would pass.
inline unsigned unit_grid(int64_t units, int per_group, int threads) {
  return (unsigned)std::min<int64_t>((units + per_group - 1) / per_group, UINT32_MAX / threads);
}

// ------------------------------------------------------------------------ scheduled dispatch
// Which form of the bf16 kernel sends `slices` slices of `pairs` pairs in all, in `chunks` 4 KiB units a row:
// the long one (four workgroups per compute unit, the next unit's loads in flight under this one's stores) or
// the short one (as many workgroups as fit, one unit at a time). A workgroup finds its slice before it
// sends, and only others on its compute unit hide that, so a slice has to be long; and with more workgroups
// than run at once their rows must not fit the 256 MB memory-side cache, or how writes spread over the memory
// does not matter. us in the long / short form: 64 ranks x 128 tokens x 7168 columns, 64 workers 211 / 268;
// 16 x 128 x 2048, 32 workers 16.4 / 17.0, 128 workers 17.2 / 15.0; 256 x 16 x 1024, 64 workers 60 / 35; 256 x
// 32 x 512, 8 workers 22.4 / 16.8; 32 x 64 x 5120, 48 workers 33.9 / 28.1.
constexpr int kLongSliceUnits = 32;
constexpr int kLongSlicesAtOnce = 1024;        // four workgroups on each of 256 compute units
constexpr int64_t kLongRowBytes = 256 << 20;
inline bool long_slices(int64_t pairs, int H, int chunks, int64_t slices) {
  return pairs * chunks >= slices * kLongSliceUnits && (slices <= kLongSlicesAtOnce || pairs * H * 2 >= kLongRowBytes);
}

// ------------------------------------------------------------------------ one-launch layers
constexpr int kFewChoices = 2;    // up to this many choices a wave has little to write, and more waves are run
constexpr int kSendBatch = 4;     // most tokens a send workgroup takes at a time: one per wave

// How the layer variants' combine learns that a row chunk has arrived (Data-as-Flag):
// kDafNone is the launch without a combine (layout and dispatch only).
constexpr int kDafNone = 0;       // no combine role
constexpr int kDafSentinel = 1;   // Sentinel Polling: every element compared with the reserved pattern
constexpr int kDafFlag = 2;       // Token-Flag Fusion: an epoch flag per 1 KiB chunk, stored after the chunk
constexpr int kDafChecksum = 3;   // Data-for-Checksum: a salted hash per 1 KiB chunk, checked against the data

// Forms of the kernel. In all but the split one every workgroup that sends goes on to combine; there the
// workgroups past the senders only combine, a row at a time.
constexpr int kFormGeneral = 0;
constexpr int kFormFew = 1;    // up to kFewChoices choices: fewer loads together, less to compile and to fetch
constexpr int kFormWide = 2;   // layout and dispatch of many long rows (see scalar_wave)
constexpr int kFormSplit = 3;

// 1 KiB units a send wave loads together. Waiting for a load that was issued behind stores is waiting for
// those stores, so a wave loads several units before it stores any. Layout and dispatch, us per layer at 2 / 4 / 6
// units: 32 ranks x 64 tokens x 7168 columns 111.4 / 108.4 / 105.7, 64 x 128 x 7168 407 / 408.5 / 407, 64 x 128 x 256 47.3 /
// 47.0 / 48.9, 64 x 256 top-4 x 1024 84.0 / 83.7 / 85.9; top-1, 32 x 1024 x 256 71.7 / 74.2 / 77.2. The split form's code is fetched anew by every compute unit, which counts in layers
// of 20 us: with 1 / 4 units ahead (24 and 29 KB of code) 512 tokens top-2 x 256 columns 16.3 / 17.0.
constexpr int send_ahead(int form, bool layer) {
  return form == kFormSplit ? 1 : form == kFormFew && !layer ? 2 : 4;
}

// Whether the send and combine roles hold the wave's index in their workgroup as a scalar, which makes the
// loads of x single instructions, or in a vector register, which makes them loops over lanes. us with the
// scalar / the vector, layout and dispatch: 64 ranks x 128 tokens x 7168 columns 409.8 / 408.3, but 64 x 256 top-4 x
// 1024 83.7 / 87, 64 x 64 top-16 x 2048 123.7 / 128, 64 x 4 x 7168 31.0 / 32.9. In the general form of the layers it is a matter of
// the shape: Sentinel, 32 x 64 x 7168 149 / 159, 16 x 128 x 2048 55.6 / 54.7, 32 x 64 top-4 x 512 27.1 / 26.8.
constexpr bool scalar_wave(int form, bool layer) {
  return form == kFormFew || form == kFormSplit || (form == kFormGeneral && !layer);
}
constexpr int kWideChunks = 8;
constexpr int64_t kWideTokens = 2048;

// Which form takes a layer. Against workgroups of their own for the combine, a whole device that sends and
// then combines has more waves for each, but places every token twice in a row and overlaps nothing. Whole
// layer, speed split / joined against the first form that this kernel had:
// * short rows in several rounds of batches: top-1, 32 ranks x 1024 tokens x 256 columns, Sentinel 1.16 / 0.85,
//   flag 1.31 / 1.08, checksum 1.15 / 1.05; top-3, 32 x 512 x 256 1.13 / 0.84, 1.21 / 1.11, 1.10 / 0.92; with two 1 KiB
//   chunks the joined form wins (top-2, 32 x 1024 x 1024, Sentinel 1.17 / 1.23);
// * few tokens: top-2, 4 x 128 x 256 1.00 / 0.84, 0.96 / 0.91, 1.01 / 0.97; top-4, 16 x 2 x 4992 0.96 / 0.76, 0.92 /
//   0.86, 0.96 / 0.80; top-8, 8 x 16 x 2048 1.15 / 0.99, 1.07 / 1.14, 1.13 / 1.04; top-8, 64 x 4 x 7168, checksum 1.15 / 0.96.
constexpr int64_t kSplitFewTokens = 512;    // and fewer than kSplitFewUnits 1 KiB chunks of rows
constexpr int64_t kSplitFewUnits = 4096;
constexpr int kSplitFlagChoices = 4;        // with more, Token-Flag Fusion is faster joined
constexpr int64_t kSplitShortTokens = 4096;  // rows of one 1 KiB chunk, more than one batch per workgroup
constexpr int kSplitShortSentinel = 8, kSplitShortMarks = 3;  // and at most this many choices
inline int joined_form(const Geom& g, int H, int sync) {
  if (g.k <= kFewChoices) return kFormFew;
  const int cchunks = (H / 8 + kWave - 1) / kWave;
  return sync == kDafNone && cchunks >= kWideChunks && g.T >= kWideTokens ? kFormWide : kFormGeneral;
}
inline int decomposed_form(const Geom& g, int H, int sync) {
  const int64_t cchunks = (H / 8 + kWave - 1) / kWave;
  if (sync != kDafNone) {
    const bool few_tokens = g.T <= kSplitFewTokens && g.T * cchunks < kSplitFewUnits &&
                            (sync != kDafFlag || g.k <= kSplitFlagChoices);
    const bool short_rows = cchunks == 1 && g.T > kSplitShortTokens &&
                            g.k <= (sync == kDafSentinel ? kSplitShortSentinel : kSplitShortMarks);
    if (few_tokens || short_rows) return kFormSplit;
  }
  return joined_form(g, H, sync);
}

// Workgroups of the launch by role, and the device's co-resident capacity for it.
struct DecomposedPlan {
  int form;
  int grid, count_groups, send_groups, capacity;
  int senders;      // workgroups that send: send_groups, or the whole grid
  int batch;        // tokens a send workgroup takes at a time
  int combine_run;  // 1 KiB column chunks per combine task
};

// Send workgroups per compute unit. Scattered writes go faster from fewer waves: layout and dispatch, us
// per layer at 2 / 3 workgroups (4 waves each): 32 ranks x 64 tokens x 7168 columns 108 / 112, 64 x 128 x
// 7168 407 / 412, 16 x 128 x 2048 44.9 / 45.0. The layer variants also combine with them, and gathers want
// more waves: at 3 / 4 workgroups 32 x 64 x 7168 168 / 158, 64 x 128 x 7168 636 / 629.
// With one or two choices a wave has little to write: more workgroups, and beyond one batch each the count
// workgroups join when they have counted (top-1 of 1024 columns on 32 ranks, us per layer without and with:
// 1024 tokens each, layout and dispatch 120 / 99; 256 tokens each, the sentinel layer 48.7 / 46.4). At 3 / 4 / 5 / 7 of
// them, layout and dispatch, top-2 x 1024 tokens x 256 columns 83.4 / 80.6 / 81.0 / 84.5, top-1 x 1024 x 4096 277 / 280 /
// 284 / 285; the Sentinel layer of top-1 x 1024 x 4096 at 4 / 5 / 6 296 / 290 / 336.
constexpr int kSendPerCu = 2, kSendPerCuLayer = 4, kSendPerCuFew = 4, kSendPerCuFewLayer = 5;

// The plan on a device of `cus` compute units that holds `capacity` workgroups of the kernel's form at once.
// A grid beyond the capacity (a count_groups that leaves no room for send workgroups) is the caller's to
// refuse; sums that would not fit an int saturate, so that such a grid is never below the capacity.
inline DecomposedPlan split_decomposed(const Geom& g, int H, int count_groups, int sync, int form, int capacity, int cus) {
  DecomposedPlan plan;
  plan.form = form;
  plan.capacity = capacity;
  // Default split: one count workgroup per layout chunk, at most a quarter of what the device
  // holds at once.
  const int64_t nc = count_groups > 0 ? count_groups : std::min(g.nblk, std::max(1, capacity / 4));
  plan.count_groups = (int)nc;
  const int64_t cchunks = (H / 8 + kWave - 1) / kWave;
  // Send: batches of up to four tokens, all workgroups with as many batches as the next.
  const bool few = g.k <= kFewChoices;
  const int most_per_cu = sync == kDafNone ? (few ? kSendPerCuFew : kSendPerCu) : few ? kSendPerCuFewLayer : kSendPerCuLayer;
  int64_t groups = std::max<int64_t>(1, std::min<int64_t>(capacity - nc, (int64_t)most_per_cu * cus));
  const int64_t room = groups + (few && form != kFormSplit && g.T > groups * kSendBatch ? nc : 0);
  const int64_t rounds = std::max<int64_t>(1, (g.T + room * kSendBatch - 1) / (room * kSendBatch));
  const int64_t even = (g.T + room * rounds - 1) / (room * rounds);
  // More tokens per batch than that where a row is so short that a wave would load fewer than four
  // units, and every wave should place a token, as long as each compute unit keeps a workgroup (128 tokens of
  // 2048 columns: one per batch 26.6 us, four 46.1); with few choices, and for rows that leave waves of the workgroup
  // idle, also when it does not: every workgroup's start and its count at the end cost as well (256 tokens top-1 of
  // 2048 columns: one per batch 16.8 us, four 15.6).
  const int64_t full = (4 * kSendBatch + cchunks - 1) / cchunks;
  int64_t batch = std::max(even, std::min(full, few && sync == kDafNone ? full : g.T / cus));
  batch = std::max<int64_t>(batch, kSendBatch / cchunks);
  plan.batch = (int)std::max<int64_t>(1, std::min<int64_t>(kSendBatch, batch));
  if (form == kFormSplit) groups = std::max<int64_t>(1, (capacity - nc) / 2);
  plan.send_groups = (int)std::max<int64_t>(1, std::min<int64_t>(groups, (g.T + plan.batch - 1) / plan.batch));
  plan.grid = (int)std::min<int64_t>(nc + plan.send_groups, INT_MAX);
  plan.senders = room > groups ? plan.grid : plan.send_groups;
  if (form == kFormSplit) {  // the rest combine, a (token, chunk) per wave at a time
    plan.senders = plan.send_groups;
    const int64_t units = (g.T * cchunks + kLayoutWaves - 1) / kLayoutWaves;
    const int64_t rest = std::max<int64_t>(1, std::min<int64_t>(capacity - nc - plan.send_groups, units));
    plan.grid = (int)std::min<int64_t>(plan.grid + rest, INT_MAX);
  }
  // Combine: as many chunks per task as leave every wave a task, in runs of even length.
  const int64_t waves = (int64_t)plan.grid * kLayoutWaves;
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>(cchunks, (g.T * cchunks + waves - 1) / waves));
  const int64_t runs = (cchunks + want - 1) / want;
  plan.combine_run = (int)((cchunks + runs - 1) / runs);
  return plan;
}

}  // namespace epl
