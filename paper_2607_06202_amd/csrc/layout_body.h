// Device bodies of the layout's counting kernels, shared by the three-launch layout
// (layout.hip: K1 route_hist, K2 route_scan) and the decomposed single-launch layer
// (decomposed.hip), where count workgroups run the same bodies with device-scope accesses to the
// data other workgroups of the same kernel read (the C template argument, see ld32/st32).
#pragma once

#include "epl_internal.h"

namespace epl {

// Dedup and stable ranks work on waves that hold whole tokens, one lane per pair: tpw = 64 / k tokens,
// lane tl * k + j for pair j of the wave's token tl. Lanes past tpw * k hold nothing.
struct PairLane {
  int tl, j;          // the lane's token within the wave, and its choice
  uint64_t of_token;  // the lanes of the same token
};
__device__ __forceinline__ PairLane pair_lane(const Geom& G) {
  PairLane P;
  const int lane = lane_id();
  P.tl = small_div(lane, G.inv_k);
  P.j = lane - P.tl * G.k;
  P.of_token = ((1ull << G.k) - 1) << (P.tl * G.k);
  return P;
}

// Zeroes n ints of LDS from a 16-byte aligned start, with a workgroup of THREADS threads.
template <int THREADS>
__device__ __forceinline__ void clear_lds(int32_t* p, int n) {
  for (int i = threadIdx.x; i < n / 4; i += THREADS) reinterpret_cast<int4*>(p)[i] = int4{0, 0, 0, 0};
  if ((int)threadIdx.x < n % 4) p[n / 4 * 4 + threadIdx.x] = 0;
}

// Waves' steps over one chunk: a wave holds at most 64 / k whole tokens at a time, and 1024 pairs over four
// waves take at most this many steps (k = 22: 46 tokens, 12 per wave, 2 at a time).
constexpr int kChunkSteps = 6;

// Workgroups are dealt to the MI355X's 8 XCDs in turn (workgroup i to XCD i % 8), and each XCD
// has its own L2. K1 and K3 take chunk xcd_chunk(i, nblk) in workgroup i, so that every XCD
// handles one contiguous eighth of the chunks (the tail past 8 * (nblk / 8) keeps i). Their
// small scattered stores then fall into whole lines in one L2: K1's per-chunk expert counts
// ([E][nblk], adjacent chunks adjacent), and K3's recv_src / recv_j (within an expert, the rows
// of adjacent chunks of a source rank are adjacent).
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_chunk(int i, int n) {
  const int per = n / kXcds;
  return i < per * kXcds ? (i % kXcds) * per + i / kXcds : i;
}

// K1 on chunk b (CT whole tokens of one source rank): LDS histograms of expert ids and of
// first-per-token destination ranks (the lowest lane of a token's lanes with the same rank, from one
// ballot per key bit), written as the chunk's row of chunk_r [nblk][R] and its expert counts:
// * without C (for K2 and K3): the chunk's column of chunk_e [E][nblk];
// * with C (the decomposed launch, device-scope stores): the chunk's row of cnt [nblk][E] (whole
//   lines: single 4-byte device-scope stores into lines other workgroups also write each cost a
//   read-modify-write of the line in memory), and fmask, each token's bitmask of first pairs.
// It also writes tok_nranks and the chunk's invalid count. lds holds E + R ints, red kLayoutWaves; the
// whole workgroup calls it.
template <bool C>
__device__ __forceinline__ void hist_chunk(const Geom& G, int b, const int32_t* __restrict__ idx,
                                           int32_t* __restrict__ tok_nranks, int32_t* __restrict__ chunk_e,
                                           int32_t* __restrict__ chunk_r, int32_t* __restrict__ inval,
                                           uint32_t* __restrict__ fmask, int32_t* lds, int32_t* red,
                                           int32_t* __restrict__ cnt = nullptr) {
  int32_t* hist_e = lds;           // [E]
  int32_t* hist_r = hist_e + G.E;  // [R]

  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int w = tid / kWave;
  const int s = b / G.NC;
  const int c = b - s * G.NC;
  const int t0 = c * G.CT;
  const int nt = max(0, min(G.CT, G.Tr - t0));
  const int64_t g0 = (int64_t)s * G.Tr + t0;
  const int tpw = kWave / G.k;
  const PairLane P = pair_lane(G);

  // Issue the global loads first; their latency overlaps the LDS clearing and the barrier.
  const int32_t* src = idx + g0 * G.k;
  int ids[kChunkSteps];
#pragma unroll
  for (int q = 0; q < kChunkSteps; ++q) {
    const int t = (q * kLayoutWaves + w) * tpw;  // the wave's first token of the step
    ids[q] = t + P.tl < nt && P.tl < tpw ? src[t * G.k + lane] : -1;
  }
  for (int i = tid; i < G.E + G.R; i += kLayoutThreads) lds[i] = 0;
  __syncthreads();

  int my_inval = 0;
#pragma unroll
  for (int q = 0; q < kChunkSteps; ++q) {
    const int t = (q * kLayoutWaves + w) * tpw;
    if (t >= nt) break;  // wave-uniform
    const bool in = t + P.tl < nt && P.tl < tpw;
    const int e = ids[q];
    const bool valid = in && (unsigned)e < (unsigned)G.E;
    const int d = valid ? small_div(e, G.inv_El) : 0;
    if (valid) atomicAdd(&hist_e[e], 1);
    my_inval += in && !valid;
    const uint64_t same = match_key(valid, d, G.rbits) & P.of_token;
    const bool first = valid && __builtin_ctzll(same) == lane;
    if (first) atomicAdd(&hist_r[d], 1);
    const uint64_t firsts = __ballot(first) & P.of_token;
    if (in && P.j == 0) {
      tok_nranks[g0 + t + P.tl] = __popcll(firsts);
      if constexpr (C) st32<C>(&fmask[g0 + t + P.tl], (uint32_t)(firsts >> lane));
    }
  }
  const int wsum = wave_sum(my_inval);
  if (lane == 0) red[w] = wsum;
  __syncthreads();

  if constexpr (C)
    for (int e = tid; e < G.E; e += kLayoutThreads) st32<C>(&cnt[(int64_t)b * G.E + e], hist_e[e]);
  else
    for (int e = tid; e < G.E; e += kLayoutThreads) chunk_e[(int64_t)e * G.nblk + b] = hist_e[e];
  for (int r = tid; r < G.R; r += kLayoutThreads) st32<C>(&chunk_r[(int64_t)b * G.R + r], hist_r[r]);
  if (tid == 0) {
    int n = 0;
    for (int i = 0; i < kLayoutWaves; ++i) n += red[i];
    st32<C>(&inval[b], n);
  }
}

// Stable ranks and rank slots of one chunk's pairs (nt tokens, the first of them g0), in the first WAVES
// waves of the calling workgroup of THREADS threads, each with a contiguous share of the tokens; STEPS
// bounds a wave's steps.
// All inputs are in LDS:
// * base_e [E]: the first packed row of this chunk's pairs of expert e;
// * base_r [R]: the first slot of this chunk's tokens bound for rank r;
// * whe/whr [WAVES][E] and [WAVES][R]: zeroed.
// Every pair gets its stable rank among equal keys of the chunk: one ballot per key bit, popcount of
// the lanes below, and per-wave LDS running counts; a cross-wave prefix then yields pair_row,
// pair_rslot, recv_src and recv_j. P is the number of valid pairs in the whole layout;
// rows at or past it are never written. load(q, t, in) returns the lane's id in the wave's step q, whose
// first token is t; it runs before anything waits. ready() runs between the ranks and their use: base_e, base_r
// and P must be there after it, and it synchronises the workgroup. NRANKS also writes tok_nranks.
template <int WAVES, int STEPS, int THREADS, bool NRANKS, class LoadFn, class ReadyFn>
__device__ __forceinline__ void assign_chunk_rows(const Geom& G, int nt, int64_t g0, LoadFn load, ReadyFn ready,
                                                  const int32_t* base_e, const int32_t* base_r, int32_t* whe,
                                                  int32_t* whr, int32_t* __restrict__ pair_row,
                                                  int32_t* __restrict__ pair_rslot, int32_t* __restrict__ recv_src,
                                                  int32_t* __restrict__ recv_j, int32_t* __restrict__ tok_nranks) {
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int w = tid / kWave;
  const int tpw = kWave / G.k;
  const int share = (nt + WAVES - 1) / WAVES;  // tokens per wave
  const int t_beg = w * share, t_end = min(nt, t_beg + share);
  const PairLane P = pair_lane(G);
  int id[STEPS], rank_e[STEPS], rank_r[STEPS], lead[STEPS];
#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    const int t = t_beg + q * tpw;
    id[q] = load(q, t, t + P.tl < t_end && P.tl < tpw);  // nothing for waves past WAVES: their t_beg >= nt
  }
  __syncthreads();  // whe and whr are zero
#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    rank_e[q] = rank_r[q] = 0;
    lead[q] = lane;
    const int t = t_beg + q * tpw;
    if (t >= t_end) continue;  // wave-uniform
    const bool in = t + P.tl < t_end && P.tl < tpw;
    const int e = id[q];
    const bool valid = in && (unsigned)e < (unsigned)G.E;
    const int ev = valid ? e : 0;
    const int d = valid ? small_div(e, G.inv_El) : 0;

    const uint64_t me = match_key(valid, ev, G.ebits);
    const int lo_e = rank_in_mask(me);
    const int seen_e = valid ? whe[w * G.E + e] : 0;
    if (valid && lo_e == 0) whe[w * G.E + e] = seen_e + __popcll(me);  // one lane per key
    rank_e[q] = seen_e + lo_e;

    const uint64_t md = match_key(valid, d, G.rbits);
    if (valid) lead[q] = (int)__builtin_ctzll(md & P.of_token);  // the token's first pair on the rank
    const bool first = valid && lead[q] == lane;
    const uint64_t firsts = __ballot(first);
    const uint64_t mr = md & firsts;
    const int lo_r = rank_in_mask(mr);
    const int seen_r = first ? whr[w * G.R + d] : 0;
    if (first && lo_r == 0) whr[w * G.R + d] = seen_r + __popcll(mr);
    rank_r[q] = seen_r + lo_r;
    if constexpr (NRANKS) {
      if (in && P.j == 0) tok_nranks[g0 + t + P.tl] = __popcll(firsts & P.of_token);
    }
  }
  const int total = ready();

  // Per-wave counts -> per-wave bases (exclusive prefix over waves, in wave order).
  for (int e = tid; e < G.E; e += THREADS) {
    int run = base_e[e];
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
      const int h = whe[v * G.E + e];
      whe[v * G.E + e] = run;
      run += h;
    }
  }
  for (int r = tid; r < G.R; r += THREADS) {
    int run = base_r[r];
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
      const int h = whr[v * G.R + r];
      whr[v * G.R + r] = run;
      run += h;
    }
  }
  __syncthreads();

#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    const int t = t_beg + q * tpw;
    if (t >= t_end) continue;
    const bool in = t + P.tl < t_end && P.tl < tpw;
    const int e = id[q];
    const bool valid = in && (unsigned)e < (unsigned)G.E;
    const int d = valid ? small_div(e, G.inv_El) : 0;
    const int row = valid ? whe[w * G.E + e] + rank_e[q] : -1;
    const int slot = valid && lead[q] == lane ? whr[w * G.R + d] + rank_r[q] : -1;
    const int rslot = __shfl(slot, lead[q], kWave);  // every pair reports its token's first pair on the rank
    if (in) {
      const int64_t p = (g0 + t) * G.k + lane;
      pair_row[p] = row;
      pair_rslot[p] = valid ? rslot : -1;
      if (valid && row < total) {  // always true for a consistent layout; keeps stores in bounds
        recv_src[row] = (int32_t)(g0 + t + P.tl);
        recv_j[row] = P.j;
      }
    }
  }
}

constexpr int kScanV = 4;  // consecutive elements per thread in one workgroup scan step

// K2 item b of E + R + 1: expert column b < E, source rank b - E < R, or the invalid total.
// scratch holds kLayoutWaves ints, seg_start EPL_MAX_EXPERTS + 1; the whole workgroup calls it.
template <bool C>
__device__ __forceinline__ void scan_item(const Geom& G, int b, int32_t* __restrict__ chunk_e,
                                          int32_t* __restrict__ chunk_r, const int32_t* __restrict__ inval,
                                          int32_t* __restrict__ recv_cnt, int32_t* __restrict__ send_cnt,
                                          int32_t* __restrict__ rank_cnt, int32_t* __restrict__ seg_rel,
                                          int32_t* __restrict__ num_invalid, int32_t* scratch, int32_t* seg_start,
                                          const int32_t* __restrict__ cnt = nullptr) {
  const int tid = threadIdx.x;
  if (b < G.E) {
    // Expert column e, laid out [source rank][chunk] (flat index s * NC + c, the order of the
    // expert's rows): an exclusive scan over the whole column gives each chunk's rows relative to
    // the expert start. The workgroup scans kScanV consecutive chunks per thread at a time; the
    // value at each rank's first chunk is that rank's segment start.
    const int e = b;
    int32_t* col = chunk_e + (int64_t)e * G.nblk;
    int carry = 0;
    for (int base = 0; base < G.nblk; base += kLayoutThreads * kScanV) {
      const int b0 = base + tid * kScanV;
      int h[kScanV];
      int sum = 0;
#pragma unroll
      for (int v = 0; v < kScanV; ++v) {
        // With C the counts come from cnt [nblk][E] (K1's rows); the bases go to chunk_e either way.
        if constexpr (C)
          h[v] = b0 + v < G.nblk ? ld32<C>(&cnt[(int64_t)(b0 + v) * G.E + e]) : 0;
        else
          h[v] = b0 + v < G.nblk ? col[b0 + v] : 0;
        sum += h[v];
      }
      int total;
      int run = carry + block_exclusive_sum(sum, total, scratch);
#pragma unroll
      for (int v = 0; v < kScanV; ++v) {
        const int bb = b0 + v;
        if (bb < G.nblk) {
          st32<C>(&col[bb], run);
          const int s = bb / G.NC;
          if (bb == s * G.NC) seg_start[s] = run;
        }
        run += h[v];
      }
      carry += total;
    }
    if (tid == 0) seg_start[G.R] = carry;
    __syncthreads();
    for (int s = tid; s < G.R; s += kLayoutThreads) {
      st32<C>(&seg_rel[e * G.R + s], seg_start[s]);
      send_cnt[s * G.E + e] = seg_start[s + 1] - seg_start[s];
    }
    if (tid == 0) st32<C>(&recv_cnt[e], carry);
  } else if (b < G.E + G.R) {
    // Source rank s: per destination rank r, slots of earlier chunks come first. The rank's
    // [chunk][R] block of counts is scanned as one flat sequence in (r, chunk) order, so each r
    // is a contiguous segment; an element's slot base is the flat exclusive prefix minus the
    // prefix at its segment's first chunk.
    const int s = b - G.E;
    int32_t* rows = chunk_r + (int64_t)s * G.NC * G.R;  // this rank's NC chunk rows of R counts
    const int n = G.NC * G.R;
    int carry = 0;
    for (int base = 0; base < n; base += kLayoutThreads * kScanV) {
      int h[kScanV], at[kScanV], rr[kScanV];
      int sum = 0;
#pragma unroll
      for (int v = 0; v < kScanV; ++v) {
        const int f = base + tid * kScanV + v;
        rr[v] = f / G.NC;
        const int c = f - rr[v] * G.NC;
        at[v] = f < n ? c * G.R + rr[v] : -1;
        h[v] = f < n ? ld32<C>(&rows[at[v]]) : 0;
        sum += h[v];
      }
      int total;
      int run = carry + block_exclusive_sum(sum, total, scratch);
      int pre[kScanV];
#pragma unroll
      for (int v = 0; v < kScanV; ++v) {
        pre[v] = run;
        if (at[v] >= 0 && at[v] < G.R) seg_start[rr[v]] = run;  // chunk 0 of rank rr[v]
        run += h[v];
      }
      carry += total;
      __syncthreads();  // segment starts found in this step are visible
#pragma unroll
      for (int v = 0; v < kScanV; ++v)
        if (at[v] >= 0) st32<C>(&rows[at[v]], pre[v] - seg_start[rr[v]]);
    }
    if (tid == 0) seg_start[G.R] = carry;
    __syncthreads();
    for (int r = tid; r < G.R; r += kLayoutThreads) rank_cnt[s * G.R + r] = seg_start[r + 1] - seg_start[r];
  } else {
    int n = 0;
    for (int i = tid; i < G.nblk; i += kLayoutThreads) n += ld32<C>(&inval[i]);
    const int w = wave_sum(n);
    if (lane_id() == 0) scratch[tid / kWave] = w;
    __syncthreads();
    if (tid == 0) {
      int t = 0;
      for (int i = 0; i < kLayoutWaves; ++i) t += scratch[i];
      num_invalid[0] = t;
    }
  }
}

}  // namespace epl
