// Routing layout for MoE dispatch on one GPU: per-(source rank, expert) histograms, CalCumSum
// prefix scans, stable packed-row assignment and per-token destination-rank dedup.
//
// The paper's dispatch reports per-expert token counts from every source. Prefix sums of those
// counts give each expert's HBM offsets, and tokens are then laid out contiguously per expert
// (Background phases 3 and 5; Kernel Decomposition: TokenCnt-Sending, CalCumSum,
// Token-Reordering). All ranks are virtual here, so the count "exchange" is just reading the
// [rank][expert] matrix by column.
//
// Three launches, no atomics that decide an order, bit-identical on every run (small layouts
// take one launch instead, route_single in small.hip, with the same outputs):
//   K1 route_hist      one workgroup per chunk (CT whole tokens of one source rank): LDS
//                      histograms of expert ids and of first-per-token destination ranks, the
//                      tok_nranks and the invalid count.
//   K2 route_scan      one workgroup per expert column: scan over (source rank, chunk) giving
//                      segment offsets relative to the expert start, send_cnt, recv_cnt and
//                      per-chunk base rows. One workgroup per source rank: scan of rank slots
//                      over chunks. One workgroup: num_invalid.
//   K3 route_finalize  one workgroup per chunk: expert_off via an LDS scan of recv_cnt. Each
//                      wave takes a contiguous quarter of the chunk's tokens and gives every pair
//                      its stable rank among equal keys: ballot match over the key bits,
//                      popcount of the lanes below, per-wave LDS running counts. A cross-wave
//                      prefix then yields pair_row, recv_src, recv_j and pair_rslot.
// For layouts of at most kPlaceMaxChunks chunks and 256 experts (place_layout) epl_layout_dispatch takes two
// launches before the rows, route_count and route_place.
//
// Small integer quotients (pair -> token within a chunk, expert -> rank, seg_off index -> expert;
// every numerator < 2^21) use small_div, which is exact in that range.
#include "layout_body.h"

namespace epl {

// ------------------------------------------------------------------------------------ K1
__global__ void __launch_bounds__(kLayoutThreads)
    route_hist_kernel(Geom G, const int32_t* __restrict__ idx, int32_t* __restrict__ tok_nranks,
                      int32_t* __restrict__ chunk_e, int32_t* __restrict__ chunk_r, int32_t* __restrict__ inval) {
  extern __shared__ int32_t lds[];
  __shared__ int32_t red[kLayoutWaves];
  hist_chunk<false>(G, xcd_chunk(blockIdx.x, G.nblk), idx, tok_nranks, chunk_e, chunk_r, inval, nullptr, lds, red);
}

// ------------------------------------------------------------------------------------ K2
__global__ void __launch_bounds__(kLayoutThreads)
    route_scan_kernel(Geom G, int32_t* __restrict__ chunk_e, int32_t* __restrict__ chunk_r,
                      const int32_t* __restrict__ inval, int32_t* __restrict__ recv_cnt, int32_t* __restrict__ send_cnt,
                      int32_t* __restrict__ rank_cnt, int32_t* __restrict__ seg_rel, int32_t* __restrict__ num_invalid) {
  __shared__ int32_t scratch[kLayoutWaves];
  __shared__ int32_t seg_start[EPL_MAX_EXPERTS + 1];  // per source rank (R <= E), then the total
  scan_item<false>(G, blockIdx.x, chunk_e, chunk_r, inval, recv_cnt, send_cnt, rank_cnt, seg_rel, num_invalid,
                   scratch, seg_start);
}

// ------------------------------------------------------------------------------------ K3
__global__ void __launch_bounds__(kLayoutThreads)
    route_finalize_kernel(Geom G, const int32_t* __restrict__ idx, const int32_t* __restrict__ chunk_e,
                          const int32_t* __restrict__ chunk_r, const int32_t* __restrict__ recv_cnt,
                          const int32_t* __restrict__ seg_rel, int32_t* __restrict__ expert_off,
                          int32_t* __restrict__ rank_off, int32_t* __restrict__ seg_off, int32_t* __restrict__ pair_row,
                          int32_t* __restrict__ pair_rslot, int32_t* __restrict__ recv_src,
                          int32_t* __restrict__ recv_j) {
  extern __shared__ int32_t lds[];
  int32_t* eoff = lds;               // [E+1]
  int32_t* base_e = eoff + G.E + 1;  // [E]   first packed row of this chunk's pairs of expert e
  int32_t* base_r = base_e + G.E;    // [R]   first slot of this chunk's tokens bound for rank r
  int32_t* whe = base_r + G.R;       // [W][E] per-wave counts, then per-wave bases
  int32_t* whr = whe + kLayoutWaves * G.E;  // [W][R]
  __shared__ int32_t scratch[kLayoutWaves];

  const int tid = threadIdx.x;
  const int b = xcd_chunk(blockIdx.x, G.nblk);
  const int s = b / G.NC;
  const int c = b - s * G.NC;
  const int t0 = c * G.CT;
  const int nt = max(0, min(G.CT, G.Tr - t0));
  const int64_t g0 = (int64_t)s * G.Tr + t0;

  // All global inputs of this workgroup are independent: issue them together. That includes
  // the first entries of this workgroup's slice of segment offsets, which are stored at the end.
  const int nseg = G.E * G.R;
  const int seg_per = (nseg + G.nblk - 1) / G.nblk;
  const int seg_i1 = min(nseg, (b + 1) * seg_per);
  constexpr int kSegSlots = 2;
  int seg_pre[kSegSlots];
#pragma unroll
  for (int q = 0; q < kSegSlots; ++q) {
    const int i = b * seg_per + tid + q * kLayoutThreads;
    seg_pre[q] = i < seg_i1 ? seg_rel[i] : 0;
  }
  // Each lane loads its chunk counts and expert totals into registers first (indices clamped, so no
  // load sits behind a branch).
  const int per = (G.E + kLayoutThreads - 1) / kLayoutThreads;  // experts per lane in the scan below
  const int e0 = min(G.E, tid * per), e1 = min(G.E, e0 + per);
  int ce_r[kLayoutSlots], cr_r[kLayoutSlots], rc_r[kLayoutSlots];
#pragma unroll
  for (int q = 0; q < kLayoutSlots; ++q) {
    const int e = tid + q * kLayoutThreads;
    ce_r[q] = chunk_e[(int64_t)min(e, G.E - 1) * G.nblk + b];
    cr_r[q] = chunk_r[(int64_t)b * G.R + min(e, G.R - 1)];
    rc_r[q] = recv_cnt[min(e0 + q, G.E - 1)];
  }
  for (int i = tid; i < kLayoutWaves * (G.E + G.R); i += kLayoutThreads) whe[i] = 0;

  const int32_t* src = idx + g0 * G.k;
  assign_chunk_rows<kLayoutWaves, kChunkSteps, kLayoutThreads, false>(
      G, nt, g0, [&](int, int t, bool in) { return in ? src[t * G.k + lane_id()] : -1; },
      [&] {
#pragma unroll
        for (int q = 0; q < kLayoutSlots; ++q) {
          const int e = tid + q * kLayoutThreads;
          if (e < G.E) base_e[e] = ce_r[q];
          if (e < G.R) base_r[e] = cr_r[q];
        }
        // expert_off = exclusive scan of recv_cnt; each lane owns the contiguous run [e0, e1).
        int sum = 0;
#pragma unroll
        for (int q = 0; q < kLayoutSlots; ++q) sum += e0 + q < e1 ? rc_r[q] : 0;
        int total;
        int run = block_exclusive_sum(sum, total, scratch);  // synchronises the workgroup
#pragma unroll
        for (int q = 0; q < kLayoutSlots; ++q) {
          if (e0 + q >= e1) break;
          eoff[e0 + q] = run;
          base_e[e0 + q] += run;
          run += rc_r[q];
        }
        if (tid == 0) eoff[G.E] = total;
        __syncthreads();
        return total;
      },
      base_e, base_r, whe, whr, pair_row, pair_rslot, recv_src, recv_j, nullptr);

  // Global offsets, off the critical path: block 0 writes expert_off and rank_off; every
  // workgroup rebases one slice of the (expert, source) segment offsets.
  if (b == 0) {
    for (int e = tid; e <= G.E; e += kLayoutThreads) expert_off[e] = eoff[e];
    for (int d = tid; d <= G.R; d += kLayoutThreads) rank_off[d] = eoff[d * G.El];
  }
#pragma unroll
  for (int q = 0; q < kSegSlots; ++q) {
    const int i = b * seg_per + tid + q * kLayoutThreads;
    if (i < seg_i1) seg_off[i] = eoff[small_div(i, G.inv_R)] + seg_pre[q];
  }
  for (int i = b * seg_per + tid + kSegSlots * kLayoutThreads; i < seg_i1; i += kLayoutThreads)
    seg_off[i] = eoff[small_div(i, G.inv_R)] + seg_rel[i];
}

// ------------------------------------------------------------------------------------ count and place
// The layout in two launches, for layouts of few chunks (place_layout): route_count writes the chunks'
// counts, and every workgroup of route_place sums the columns of that matrix itself, up to the chunk's
// source rank, up to the chunk and in all, which gives what K2 would have written for it.
// What bounds it is the matrix, which every compute unit reads through the L2 (41 bytes per ns each: 3.1 us
// for the 256 rows of a 256-chunk layout), and then instructions. So counts are 16 bits, eight of them to a
// lane's load, and route_count also writes the sum of every kGroupChunks chunks: route_place reads those
// and the few single chunks between them and the two places where it splits the columns. A thread's
// sums stay in pairs of 16-bit halves until the workgroup adds them up (place_layout bounds them), and the
// workgroup has four waves: sixteen, with a quarter of the loads each, took longer to start, to meet and
// to add up (8.2 us at 256 chunks).
constexpr int kCountThreads = 1024;
constexpr int kGroupWaves = kCountThreads / kWave / kGroupChunks;  // waves of route_count per chunk

// One workgroup per kGroupChunks chunks, four waves each: the chunks' rows of cnt and the group's row of
// group_cnt, [(E+1)/2] words of two 16-bit expert counts, and the chunks' rows of chunk_r [nblk][R].
__global__ void __launch_bounds__(kCountThreads)
    route_count_kernel(Geom G, const int32_t* __restrict__ idx, int32_t* __restrict__ cnt,
                       int32_t* __restrict__ group_cnt, int32_t* __restrict__ chunk_r) {
  extern __shared__ __align__(16) int32_t lds[];  // [kGroupChunks][E + R]
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int i = tid / kWave / kGroupWaves;  // the wave's chunk of the group
  const int w = tid / kWave % kGroupWaves;
  const int b = (int)blockIdx.x * kGroupChunks + i;
  const int s = b / G.NC;
  const int t0 = (b - s * G.NC) * G.CT;
  const int nt = b < G.nblk ? max(0, min(G.CT, G.Tr - t0)) : 0;
  const int tpw = kWave / G.k;
  const PairLane P = pair_lane(G);
  const int32_t* src = idx + ((int64_t)s * G.Tr + t0) * G.k;
  int32_t* hist_e = lds + i * (G.E + G.R);
  int32_t* hist_r = hist_e + G.E;
  int ids[kChunkSteps];
#pragma unroll
  for (int q = 0; q < kChunkSteps; ++q) {
    const int t = (q * kGroupWaves + w) * tpw;
    ids[q] = t + P.tl < nt && P.tl < tpw ? src[t * G.k + lane] : -1;
  }
  clear_lds<kCountThreads>(lds, kGroupChunks * (G.E + G.R));
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kChunkSteps; ++q) {
    const int t = (q * kGroupWaves + w) * tpw;
    if (t >= nt) break;  // wave-uniform
    const int e = ids[q];
    const bool valid = t + P.tl < nt && P.tl < tpw && (unsigned)e < (unsigned)G.E;
    const int d = valid ? small_div(e, G.inv_El) : 0;
    if (valid) atomicAdd(&hist_e[e], 1);
    const uint64_t same = match_key(valid, d, G.rbits) & P.of_token;
    if (valid && __builtin_ctzll(same) == lane) atomicAdd(&hist_r[d], 1);
  }
  __syncthreads();
  const int words = (G.E + 1) / 2;
  const int team = tid % (kWave * kGroupWaves);
  if (b < G.nblk) {
    for (int j = team; j < words; j += kWave * kGroupWaves)
      cnt[(int64_t)b * words + j] = hist_e[2 * j] | (2 * j + 1 < G.E ? hist_e[2 * j + 1] << 16 : 0);
    for (int r = team; r < G.R; r += kWave * kGroupWaves) chunk_r[(int64_t)b * G.R + r] = hist_r[r];
  }
  for (int j = tid; j < words; j += kCountThreads) {
    int lo = 0, hi = 0;
#pragma unroll
    for (int v = 0; v < kGroupChunks; ++v) {  // the last group's missing chunks counted nothing
      lo += lds[v * (G.E + G.R) + 2 * j];
      hi += 2 * j + 1 < G.E ? lds[v * (G.E + G.R) + 2 * j + 1] : 0;
    }
    group_cnt[(int64_t)blockIdx.x * words + j] = lo | hi << 16;
  }
}

// LDS word of expert e's count, so that the lanes of a wave, eight experts apart, hit consecutive words.
__device__ __forceinline__ int place_slot(int e) { return (e & 7) * kPlaceLanes + (e >> 3); }

// STEPS bounds the four waves' steps through the chunk. It writes recv_src and recv_j as well, 4 bytes to
// scattered rows; left to the row kernel's waves, among their row stores, they delayed those (layout, dispatch and
// combine, us here / there: 64 ranks x 128 tokens x 2048 columns 112.1 / 115.5, x 7168 373.9 / 375.7; 32 x 4096 top-1 x
// 128 100.3 / 102.6; 32 x 128 x 4096 111.6 / 115.2).
template <int STEPS>
__global__ void __launch_bounds__(kLayoutThreads)
    route_place_kernel(Geom G, const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt,
                       const int32_t* __restrict__ group_cnt, const int32_t* __restrict__ chunk_r,
                       epl_layout_buffers L) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  extern __shared__ __align__(16) int32_t lds[];
  // Counts of the groups before the source rank's, from there to the chunk's, and from it on; of the
  // single chunks up to the rank, and up to the chunk.
  enum { kBefore, kBetween, kRest, kToRank, kToChunk, kParts };
  int32_t* h = lds;                              // [kParts][kPlaceExperts]
  int32_t* base_r = h + kParts * kPlaceExperts;  // [R] first slot of this chunk's tokens bound for rank r
  int32_t* own_r = base_r + G.R;                 // [R] the source rank's tokens bound for rank r (its last chunk only)
  int32_t* whe = own_r + G.R;                    // [W][E]
  int32_t* whr = whe + kLayoutWaves * G.E;       // [W][R]
  int32_t* eoff = whr + kLayoutWaves * G.R;      // [E+1]
  int32_t* base_e = eoff + G.E + 1;              // [E]
  __shared__ int32_t scratch[kLayoutWaves];

  const int tid = threadIdx.x;
  const int b = xcd_chunk(blockIdx.x, G.nblk);
  const int s = b / G.NC;
  const int c = b - s * G.NC;
  const int t0 = c * G.CT;
  const int nt = max(0, min(G.CT, G.Tr - t0));
  const int64_t g0 = (int64_t)s * G.Tr + t0;
  const int rank0 = s * G.NC;  // the source rank's first chunk
  const bool last = c == G.NC - 1;
  const int groups = (G.nblk + kGroupChunks - 1) / kGroupChunks;
  const int group_a = rank0 / kGroupChunks, group_b = b / kGroupChunks;

  // The counts are in flight before anything waits; the ids follow at once, in assign_chunk_rows.
  const int32_t* src = idx + g0 * G.k;
  const int nslot = (last ? G.NC : c) * G.R;
  const int32_t* slots = chunk_r + (int64_t)rank0 * G.R;
  const int slot0 = tid < nslot ? slots[tid] : 0;
  const int words = (G.E + 1) / 2;
  const int quad = tid % kPlaceLanes;  // words [4 * quad, 4 * quad + 4) of a row; past its end they belong to no expert
  const int row = tid / kPlaceLanes;
  const int word0 = min(4 * quad, words - 1);
  u32x4 gv[kPlaceAhead], sv = {0, 0, 0, 0};
  auto load_groups = [&](int r0) {
#pragma unroll
    for (int q = 0; q < kPlaceAhead; ++q)
      __builtin_memcpy(&gv[q], group_cnt + (int64_t)min(r0 + q * kPlaceRows + row, groups - 1) * words + word0, 16);
  };
  load_groups(0);
  // The thread's single chunk, if any: rows 0-2 up to the rank, rows 3-5 up to the chunk.
  constexpr int kSingle = kGroupChunks - 1;
  const int single = row < kSingle ? group_a * kGroupChunks + row : group_b * kGroupChunks + row - kSingle;
  const bool to_rank = row < kSingle && single < rank0;
  const bool to_chunk = row >= kSingle && row < 2 * kSingle && single < b;
  if (to_rank || to_chunk) __builtin_memcpy(&sv, cnt + (int64_t)single * words + word0, 16);
  clear_lds<kLayoutThreads>(lds, kParts * kPlaceExperts + 2 * G.R + kLayoutWaves * (G.E + G.R));
  int total = 0;
  assign_chunk_rows<kLayoutWaves, STEPS, kLayoutThreads, true>(
      G, nt, g0, [&](int, int t, bool in) { return in ? src[t * G.k + lane_id()] : -1; },
      [&] {  // the ranks were worked out while the counts were in flight
        u16x2 part[3][4] = {};
        for (int r0 = 0; r0 < groups; r0 += kPlaceAhead * kPlaceRows) {
          if (r0 > 0) load_groups(r0);
#pragma unroll
          for (int q = 0; q < kPlaceAhead; ++q) {
            const int r = r0 + q * kPlaceRows + row;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint32_t u = r < groups ? gv[q][i] : 0u;
              part[kBefore][i] += __builtin_bit_cast(u16x2, r < group_a ? u : 0u);
              part[kBetween][i] += __builtin_bit_cast(u16x2, r >= group_a && r < group_b ? u : 0u);
              part[kRest][i] += __builtin_bit_cast(u16x2, r >= group_b ? u : 0u);
            }
          }
        }
        int32_t* hs = h + (to_rank ? kToRank : kToChunk) * kPlaceExperts;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const int e = 2 * (4 * quad + i) + half;
            if (e >= G.E) break;
            const int at = place_slot(e);
#pragma unroll
            for (int p = 0; p < 3; ++p) atomicAdd(&h[p * kPlaceExperts + at], (int)part[p][i][half]);
            if (to_rank || to_chunk) atomicAdd(&hs[at], half ? (int)(sv[i] >> 16) : (int)(sv[i] & 0xFFFFu));
          }
        }
        // Slots of the source rank's chunks: the earlier ones are the base, all of them rank_cnt.
        for (int i = tid; i < nslot; i += kLayoutThreads) {
          const int cc = small_div(i, G.inv_R);
          const int n = i == tid ? slot0 : slots[i];
          if (cc < c) atomicAdd(&base_r[i - cc * G.R], n);
          if (last) atomicAdd(&own_r[i - cc * G.R], n);
        }
        __syncthreads();
        // expert_off = exclusive scan of the totals, one expert per thread.
        const int at = place_slot(tid);
        const int early = h[kBefore * kPlaceExperts + at] + h[kBetween * kPlaceExperts + at];
        const int lead = early + h[kToChunk * kPlaceExperts + at];  // the expert's pairs before the chunk
        const int start = block_exclusive_sum(tid < G.E ? early + h[kRest * kPlaceExperts + at] : 0, total, scratch);
        if (tid < G.E) {
          eoff[tid] = start;
          base_e[tid] = start + lead;
        }
        if (tid == 0) eoff[G.E] = total;
        __syncthreads();
        return total;
      },
      base_e, base_r, whe, whr, L.pair_row, L.pair_rslot, L.recv_src, L.recv_j, L.tok_nranks);

  // Per-layout and per-rank outputs, each written by one workgroup.
  if (b == 0) {
    for (int e = tid; e <= G.E; e += kLayoutThreads) L.expert_off[e] = eoff[e];
    for (int d = tid; d <= G.R; d += kLayoutThreads) L.rank_off[d] = eoff[d * G.El];
    if (tid == 0) L.num_invalid[0] = (int)(G.T * G.k) - total;
  }
  if (last) {
    for (int e = tid; e < G.E; e += kLayoutThreads) {
      const int at = place_slot(e);
      const int to_rank_e = h[kBefore * kPlaceExperts + at] + h[kToRank * kPlaceExperts + at];
      L.seg_off[e * G.R + s] = eoff[e] + to_rank_e;
      // The rank's pairs of the expert: those of its earlier chunks and of this one.
      const uint32_t own = (uint32_t)cnt[(int64_t)b * words + e / 2];
      L.send_cnt[s * G.E + e] = base_e[e] - eoff[e] - to_rank_e + (int)((e & 1) ? own >> 16 : own & 0xFFFFu);
    }
    for (int r = tid; r < G.R; r += kLayoutThreads) L.rank_cnt[s * G.R + r] = own_r[r];
  }
}

// ------------------------------------------------------------------------------------ host
static size_t finalize_lds_bytes(const Geom& g) {
  return sizeof(int32_t) * ((size_t)(g.E + 1) + g.E + g.R + (size_t)kLayoutWaves * (g.E + g.R));
}

hipError_t launch_layout_place(const Geom& geom, const int32_t* idx, int32_t* ws, const epl_layout_buffers& L,
                               hipStream_t stream) {
  if (!place_layout(geom)) return hipErrorInvalidValue;  // its callers ask first
  const WsLayout wl = ws_layout(geom);
  const Geom g = place_geom(geom);
  int32_t* cnt = ws + wl.cnt;
  int32_t* group_cnt = ws + wl.chunk_e;
  int32_t* chunk_r = ws + wl.chunk_r;
  hipLaunchKernelGGL(route_count_kernel, dim3((g.nblk + kGroupChunks - 1) / kGroupChunks), dim3(kCountThreads),
                     sizeof(int32_t) * kGroupChunks * ((size_t)g.E + g.R), stream, g, idx, cnt, group_cnt, chunk_r);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  // A chunk of at most 256 pairs takes a wave at most 2 steps of at most 64 / k whole tokens.
  const bool few = g.CT * g.k <= kLayoutThreads;
  const size_t lds = sizeof(int32_t) * ((size_t)5 * kPlaceExperts + 2 * g.R + (size_t)kLayoutWaves * (g.E + g.R) +
                                        2 * g.E + 1);
  const dim3 grid(g.nblk), block(kLayoutThreads);
  if (few)
    hipLaunchKernelGGL(route_place_kernel<2>, grid, block, lds, stream, g, idx, cnt, group_cnt, chunk_r, L);
  else
    hipLaunchKernelGGL(route_place_kernel<kChunkSteps>, grid, block, lds, stream, g, idx, cnt, group_cnt, chunk_r, L);
  return hipGetLastError();
}

hipError_t launch_layout(const Geom& g, const int32_t* idx, int32_t* ws, int32_t* send_cnt, int32_t* rank_cnt,
                         int32_t* expert_off, int32_t* rank_off, int32_t* seg_off, int32_t* tok_nranks,
                         int32_t* pair_row, int32_t* pair_rslot, int32_t* recv_src, int32_t* recv_j,
                         int32_t* num_invalid, hipStream_t stream) {
  if (layout_single(g)) {
    const epl_layout_buffers L{send_cnt, rank_cnt, expert_off, rank_off, seg_off, tok_nranks,
                               pair_row, pair_rslot, recv_src, recv_j, num_invalid};
    return launch_small_layout(g, idx, L, stream);
  }
  hipError_t err = launch_layout_counts(g, idx, ws, send_cnt, rank_cnt, tok_nranks, num_invalid, stream);
  if (err != hipSuccess) return err;
  return launch_layout_finalize(g, idx, ws, expert_off, rank_off, seg_off, pair_row, pair_rslot, recv_src, recv_j,
                                stream);
}

hipError_t launch_layout_finalize(const Geom& g, const int32_t* idx, int32_t* ws, int32_t* expert_off,
                                  int32_t* rank_off, int32_t* seg_off, int32_t* pair_row, int32_t* pair_rslot,
                                  int32_t* recv_src, int32_t* recv_j, hipStream_t stream) {
  const WsLayout wl = ws_layout(g);
  hipLaunchKernelGGL(route_finalize_kernel, dim3(g.nblk), dim3(kLayoutThreads), finalize_lds_bytes(g), stream, g,
                     idx, ws + wl.chunk_e, ws + wl.chunk_r, ws + wl.recv_cnt, ws + wl.seg_rel, expert_off, rank_off,
                     seg_off, pair_row, pair_rslot, recv_src, recv_j);
  return hipGetLastError();
}

hipError_t launch_layout_counts(const Geom& g, const int32_t* idx, int32_t* ws, int32_t* send_cnt, int32_t* rank_cnt,
                                int32_t* tok_nranks, int32_t* num_invalid, hipStream_t stream) {
  const WsLayout wl = ws_layout(g);
  int32_t* chunk_e = ws + wl.chunk_e;
  int32_t* chunk_r = ws + wl.chunk_r;
  int32_t* recv_cnt = ws + wl.recv_cnt;
  int32_t* inval = ws + wl.inval;
  int32_t* seg_rel = ws + wl.seg_rel;

  const size_t lds1 = sizeof(int32_t) * ((size_t)g.E + g.R);
  hipLaunchKernelGGL(route_hist_kernel, dim3(g.nblk), dim3(kLayoutThreads), lds1, stream, g, idx, tok_nranks,
                     chunk_e, chunk_r, inval);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;

  hipLaunchKernelGGL(route_scan_kernel, dim3(g.E + g.R + 1), dim3(kLayoutThreads), 0, stream, g, chunk_e, chunk_r,
                     inval, recv_cnt, send_cnt, rank_cnt, seg_rel, num_invalid);
  return hipGetLastError();
}

}  // namespace epl
