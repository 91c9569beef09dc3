// Small layouts in one launch, alone or together with the dispatch of their rows.
//
// Up to kSingleMaxPairs pairs, what bounds a layout is the chain of launches and memory round
// trips, not its bytes. So there are no phases that hand counts over through memory: every
// workgroup takes one group of tokens of one source rank (at most 64 pairs, one wave), counts all
// T*k ids itself, and knows its pairs' rows after one pass:
// * a pass over all ids fills LDS histograms, split at the group's first pair: the pairs of each
//   expert before the group (their row base within the expert) and from the group on (with the
//   first, the expert totals, whose prefix sums are expert_off);
// * the source rank's earlier tokens are deduplicated per destination rank, one lane per pair (the
//   lanes of a token that hold the same rank, from one ballot per key bit), which gives the group's
//   slot bases;
// * one wave then ranks the group's own pairs with the same ballots, and writes their metadata.
// With SEND the workgroup goes on to copy (bf16) or quantise (fp8) its own tokens into their rows.
// The loads of its first tokens are issued before the counting and are in flight meanwhile.
// One further workgroup per source rank writes the outputs that belong to a rank (send_cnt,
// rank_cnt, its column of seg_off); the first of them also the global ones. They come first in the
// grid, beside the groups instead of after them.
//
// Whole layer with the combine, prepared calls, against a one-launch layout whose workgroups walked
// each token's choices one after another in LDS, followed by the dispatch kernel: 1K pairs on 4 ranks
// 12.2 -> 8.8 us, 1K pairs on 16 ranks 16.7 -> 9.2 us, 16K pairs of 2048 columns 40.2 -> 35.4 us;
// 4.7K pairs of 5120 columns through the plain calls 47.4 -> 41.5 us. With the same layout but the
// dispatch as a second launch these take 12.9, 12.9, 38.7 and 44.0 us; small_dispatch says which layers do.
#include "rows_body.h"

namespace epl {

static_assert(kDispatchThreads == kLayoutThreads, "block_exclusive_sum assumes layout-sized workgroups");
constexpr int kSmallVecs = 4;  // 16-byte id loads in flight per lane in the pass over all ids
constexpr int kSendNone = 0, kSendBf16 = 1, kSendFp8 = 2;

struct SmallArgs {
  Geom G;
  int GT, NG;  // tokens per group (GT * k <= 64) and groups per source rank
  int tpw;     // whole tokens per wave: 64 / k
  const int32_t* idx;
  epl_layout_buffers L;
  const u32x4* x;
  u32x4* recv;
  float* recv_scale;
  int H, pv, chunks;  // recv row pitch in 16-byte vectors, column chunks (fp8: passes) per row
  int64_t cap;
};

// Adds pair i of idx[0, n) to the histogram h[part * E + e], part = (i >= a) + (i >= b); returns this
// lane's count of ids outside [0, E). 16-byte loads when the id array is aligned for them.
__device__ __forceinline__ int count_pairs(const int32_t* __restrict__ idx, int n, int E, int a, int b, int32_t* h) {
  int inval = 0;
  auto add = [&](int i, int e) {
    if ((unsigned)e < (unsigned)E)
      atomicAdd(&h[e + (i >= a ? E : 0) + (i >= b ? E : 0)], 1);
    else
      ++inval;
  };
  int done = 0;
  if ((reinterpret_cast<uintptr_t>(idx) & 15) == 0) {
    const int nvec = n / 4;
    const int4* idx4 = reinterpret_cast<const int4*>(idx);
    for (int v0 = threadIdx.x; v0 < nvec; v0 += kLayoutThreads * kSmallVecs) {
      int4 q[kSmallVecs];
#pragma unroll
      for (int u = 0; u < kSmallVecs; ++u) q[u] = idx4[min(v0 + u * kLayoutThreads, nvec - 1)];
#pragma unroll
      for (int u = 0; u < kSmallVecs; ++u) {
        const int v = v0 + u * kLayoutThreads;
        if (v >= nvec) break;
        add(4 * v, q[u].x);
        add(4 * v + 1, q[u].y);
        add(4 * v + 2, q[u].z);
        add(4 * v + 3, q[u].w);
      }
    }
    done = nvec * 4;
  }
  for (int i = done + (int)threadIdx.x; i < n; i += kLayoutThreads) add(i, idx[i]);
  return inval;
}

// first[d] += the tokens among src's first nt that have a valid pair on destination rank d. Each
// wave takes tpw whole tokens at a time, one lane per pair; a pair counts if it is the lowest lane
// of its token with its rank. MERGE adds once per wave and rank: with one or two (rank, choice) combinations
// most lanes of a wave would add to one word, and adds to one LDS word are served one after another (layout of
// 4096 tokens, top-1 on one rank: 11.1 us -> 8.3; with more ranks or choices the ballot costs more than it saves,
// 16384 tokens on 4 ranks 11.8 -> 12.7).
constexpr int kMergeMax = 2;  // R * k
template <bool MERGE>
__device__ __forceinline__ void count_first_pairs(const SmallArgs& A, const int32_t* __restrict__ src, int nt,
                                                  int32_t* first) {
  constexpr int kAhead = 4;  // loads in flight
  const Geom& G = A.G;
  const int lane = lane_id();
  const int tl = small_div(lane, G.inv_k);
  const uint64_t mine = ((1ull << G.k) - 1) << (tl * G.k);
  const int step = A.tpw * G.k, np = nt * G.k;
  const bool in = lane < step;
  for (int p0 = (threadIdx.x / kWave) * step; p0 < np; p0 += kAhead * kLayoutWaves * step) {
    int e[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) e[q] = src[min(p0 + q * kLayoutWaves * step + lane, np - 1)];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int p = p0 + q * kLayoutWaves * step;
      if (p >= np) break;  // wave-uniform
      const bool valid = in && p + lane < np && (unsigned)e[q] < (unsigned)G.E;
      const int d = valid ? small_div(e[q], G.inv_El) : 0;
      const uint64_t same = match_key(valid, d, G.rbits);
      const bool is_first = valid && __builtin_ctzll(same & mine) == lane;
      if constexpr (MERGE) {
        const uint64_t firsts = same & __ballot(is_first);
        if (is_first && __builtin_ctzll(firsts) == lane) atomicAdd(&first[d], __popcll(firsts));
      } else if (is_first) {
        atomicAdd(&first[d], 1);
      }
    }
  }
}

// One lane per pair of the group (np <= 64 pairs of whole tokens, ids e): every output of the pair,
// and its row (-1 if invalid).
__device__ __forceinline__ int place_group(const SmallArgs& A, int64_t g0, int np, int e, const int32_t* eoff,
                                           const int32_t* before, const int32_t* first) {
  const Geom& G = A.G;
  const int lane = lane_id();
  const bool valid = lane < np && (unsigned)e < (unsigned)G.E;
  const int ev = valid ? e : 0;
  const int d = valid ? small_div(e, G.inv_El) : 0;
  const int tl = small_div(lane, G.inv_k);
  const uint64_t mine = ((1ull << G.k) - 1) << (tl * G.k);
  const uint64_t same_e = match_key(valid, ev, G.ebits);
  const uint64_t same_d = match_key(valid, d, G.rbits);
  const int lead = valid ? (int)__builtin_ctzll(same_d & mine) : lane;  // the token's first pair on its rank
  const bool is_first = valid && lead == lane;
  const uint64_t firsts = __ballot(is_first);
  const int slot = is_first ? first[d] + rank_in_mask(same_d & firsts) : -1;
  const int rslot = __shfl(slot, lead, kWave);
  const int row = valid ? eoff[ev] + before[ev] + rank_in_mask(same_e) : -1;
  if (lane < np) {
    const int64_t p = g0 * G.k + lane;
    A.L.pair_row[p] = row;
    A.L.pair_rslot[p] = valid ? rslot : -1;
    if (valid && row < eoff[G.E]) {  // always true for a consistent layout; keeps stores in bounds
      A.L.recv_src[row] = (int32_t)(g0 + tl);
      A.L.recv_j[row] = lane - tl * G.k;
    }
    if (lane == tl * G.k) A.L.tok_nranks[g0 + tl] = __popcll(firsts & mine);
  }
  return row;
}

template <int SEND, int VPL, bool MERGE>
__global__ void __launch_bounds__(kLayoutThreads) route_single_kernel(SmallArgs A) {
  extern __shared__ int32_t lds[];
  __shared__ int32_t scratch[kLayoutWaves];
  __shared__ int32_t rows_lds[kWave];
  const Geom& G = A.G;
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int w = tid / kWave;
  int32_t* h = lds;              // [3][E] pair counts before, in and after the workgroup's range
  int32_t* first = h + 3 * G.E;  // [R] first pairs of the rank's earlier tokens (all tokens for a rank's workgroup)
  int32_t* eoff = first + G.R;   // [E+1]
  const bool meta = (int)blockIdx.x < G.R;
  const int b = (int)blockIdx.x - G.R;
  const int s = meta ? (int)blockIdx.x : b / A.NG;
  const int t0 = meta ? 0 : (b - s * A.NG) * A.GT;
  const int nt = meta ? G.Tr : min(A.GT, G.Tr - t0);
  const int np = nt * G.k;
  const int64_t g0 = (int64_t)s * G.Tr + t0;
  const int n = (int)(G.T * G.k);  // <= kSingleMaxPairs
  const int a0 = (int)(g0 * G.k);
  const int32_t* rank_ids = A.idx + (int64_t)s * G.Tr * G.k;

  // The group's own ids and the wave's first piece of x are loaded before anything waits.
  const int my_id = !meta && w == 0 ? A.idx[a0 + min(lane, np - 1)] : -1;
  const int units = SEND != kSendNone && !meta ? nt * A.chunks : 0;
  const int nv = A.H / 8;
  u32x4 buf[VPL];
  auto load_unit = [&](int u, u32x4* to) {
    const int tl = u / A.chunks;
    const int v0 = (u - tl * A.chunks) * (kWave * VPL) + lane;
    const u32x4* xr = A.x + (g0 + tl) * nv;
#pragma unroll
    for (int q = 0; q < VPL; ++q) to[q] = xr[min(v0 + q * kWave, nv - 1)];
  };
  if (SEND == kSendBf16 && w < units) load_unit(w, buf);

  for (int i = tid; i < 3 * G.E + G.R; i += kLayoutThreads) lds[i] = 0;
  __syncthreads();
  const int inval = count_pairs(A.idx, n, G.E, a0, meta ? a0 + np : n, h);
  count_first_pairs<MERGE>(A, rank_ids, meta ? G.Tr : t0, first);
  __syncthreads();
  {
    const int per = (G.E + kLayoutThreads - 1) / kLayoutThreads;
    const int e0 = min(G.E, tid * per), e1 = min(G.E, e0 + per);
    int sum = 0;
    for (int e = e0; e < e1; ++e) sum += h[e] + h[G.E + e] + h[2 * G.E + e];
    int total;
    int run = block_exclusive_sum(sum, total, scratch);  // synchronises the workgroup
    for (int e = e0; e < e1; ++e) {
      eoff[e] = run;
      run += h[e] + h[G.E + e] + h[2 * G.E + e];
    }
    if (tid == 0) eoff[G.E] = total;
  }
  if (meta) {
    const int bad = wave_sum(inval);
    if (lane == 0) scratch[w] = bad;
    __syncthreads();
    for (int e = tid; e < G.E; e += kLayoutThreads) {
      A.L.send_cnt[s * G.E + e] = h[G.E + e];
      A.L.seg_off[e * G.R + s] = eoff[e] + h[e];
    }
    for (int r = tid; r < G.R; r += kLayoutThreads) A.L.rank_cnt[s * G.R + r] = first[r];
    if (s == 0) {
      for (int e = tid; e <= G.E; e += kLayoutThreads) A.L.expert_off[e] = eoff[e];
      for (int r = tid; r <= G.R; r += kLayoutThreads) A.L.rank_off[r] = eoff[r * G.El];
      if (tid == 0) A.L.num_invalid[0] = scratch[0] + scratch[1] + scratch[2] + scratch[3];
    }
    return;
  }
  __syncthreads();
  if (w == 0) rows_lds[lane] = place_group(A, g0, np, my_id, eoff, h, first);
  if constexpr (SEND == kSendNone) return;
  __syncthreads();
  if constexpr (SEND == kSendBf16) {
    for (int u = w; u < units; u += kLayoutWaves) {
      const int tl = u / A.chunks;
      const int v0 = (u - tl * A.chunks) * (kWave * VPL) + lane;
      u32x4 next[VPL];
      if (u + kLayoutWaves < units) load_unit(u + kLayoutWaves, next);  // in flight under this unit's stores
      const int my_row = lane < G.k ? rows_lds[tl * G.k + lane] : -1;
#pragma unroll
      for (int q = 0; q < VPL; ++q) {
        const int v = v0 + q * kWave;
        for (int j = 0; j < G.k; ++j) {
          const int row = __builtin_amdgcn_readlane(my_row, j);
          if (row < 0 || row >= A.cap) continue;
          if (v < nv) store_row_policy<kCachePolicySc1>(buf[q], A.recv + (int64_t)row * A.pv, nv, v);
        }
      }
#pragma unroll
      for (int q = 0; q < VPL; ++q) buf[q] = next[q];
    }
  } else if constexpr (SEND == kSendFp8) {
    for (int u = w; u < units; u += kLayoutWaves) {
      const int tl = u / A.chunks;
      dispatch_fp8_unit(A.x, [&] { return lane < G.k ? rows_lds[tl * G.k + lane] : -1; }, A.recv, A.recv_scale,
                        g0 + tl, u - tl * A.chunks, G.k, A.H, A.pv, A.cap, lane);
    }
  }
}

// ------------------------------------------------------------------------------------ host
// With fewer 4 KiB pieces than this the pieces are 1 KiB, so that every wave of the few groups has
// one (128 tokens of 2048 columns, whole layer: 9.2 us against 10.8).
constexpr int64_t kSmallWideUnits = 512;

// pieces: a row's 4 KiB chunks (fp8: passes) that the groups send, 0 for the layout alone.
static SmallArgs small_args(const Geom& g, const int32_t* idx, const epl_layout_buffers& L, int pieces) {
  SmallArgs A{};
  A.G = g;
  A.tpw = kWave / g.k;
  A.GT = group_tokens(g, pieces);
  A.NG = (g.Tr + A.GT - 1) / A.GT;
  A.idx = idx;
  A.L = L;
  return A;
}

static size_t small_lds(const Geom& g) { return sizeof(int32_t) * ((size_t)4 * g.E + g.R + 1); }

template <int SEND, int VPL>
static hipError_t launch_single(const SmallArgs& A, hipStream_t stream) {
  const Geom& g = A.G;
  const dim3 grid(g.R * (1 + A.NG)), block(kLayoutThreads);
  if (g.R * g.k <= kMergeMax)
    hipLaunchKernelGGL((route_single_kernel<SEND, VPL, true>), grid, block, small_lds(g), stream, A);
  else
    hipLaunchKernelGGL((route_single_kernel<SEND, VPL, false>), grid, block, small_lds(g), stream, A);
  return hipGetLastError();
}

hipError_t launch_small_layout(const Geom& g, const int32_t* idx, const epl_layout_buffers& L, hipStream_t stream) {
  return launch_single<kSendNone, 1>(small_args(g, idx, L, 0), stream);
}

hipError_t launch_small_layout_dispatch(const Geom& g, const int32_t* idx, const epl_layout_buffers& L, const void* x,
                                        void* recv, float* recv_scale, int H, int pitch, int64_t cap, bool fp8,
                                        hipStream_t stream) {
  const int nv = H / 8;
  static_assert(kBf16Cols * 8 == 2048, "small_pieces counts pieces of 2048 columns");
  const int pieces = small_pieces(H, fp8);
  SmallArgs A = small_args(g, idx, L, pieces);
  A.x = static_cast<const u32x4*>(x);
  A.recv = static_cast<u32x4*>(recv);
  A.recv_scale = recv_scale;
  A.H = H;
  A.pv = fp8 ? pitch / 16 : pitch / 8;
  A.chunks = pieces;
  A.cap = cap;
  if (fp8) return launch_single<kSendFp8, 1>(A, stream);
  if (g.T * pieces >= kSmallWideUnits) return launch_single<kSendBf16, kBf16VPL>(A, stream);
  A.chunks = (nv + kWave - 1) / kWave;
  return launch_single<kSendBf16, 1>(A, stream);
}

}  // namespace epl
