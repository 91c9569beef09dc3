// Layout and dispatch in one launch, decomposed into count and send workgroups (the paper's
// Kernel Decomposition, with its point-to-point synchronisation in place of global barriers).
//
// epl_layout_dispatch runs the layout's counts, its placement and then the row kernel (layout.hip,
// dispatch.hip), with a kernel boundary between each. Here one launch holds both roles, with the bodies of
// the three-launch layout's histogram (K1) and scan (K2), as the paper splits an NPU's vector cores into a group that counts tokens and computes
// the prefix sums and a group that sends tokens:
//   * count workgroups [0, nc) run K1 on chunks i, i + nc, ..., meet at a counter (every count
//     workgroup has finished its chunks), run the K2 items i, i + nc, ..., and count themselves
//     again; the last one publishes the ready word. They then write the expert, rank and segment
//     offsets (one slice each);
//   * send workgroups [nc, grid) issue the loads of their first tokens, wait for the ready word,
//     and then place and send batches of tokens, striding over them;
//   * in the layer variants every workgroup then combines (Data-as-Flag, below), or, in the split form, the
//     workgroups past the senders combine meanwhile (geometry.h says which layers take which form).
// The count/send split nc is the knob the paper sizes by its latency model (count cores in
// proportion to the experts and inversely to the token load).
//
// Synchronisation on MI355X. Every word that one workgroup writes and another reads inside the
// launch is written with device-scope stores (ld32/st32 with C set), which need no cache
// write-back; the count role writes its per-chunk expert counts chunk-major (cnt, one contiguous
// row per chunk), because single 4-byte device-scope stores into lines that other workgroups also
// write each cost a read-modify-write in memory. A workgroup publishes by waiting for its own
// stores to complete (vmcnt), then adding to a counter with a device-scope atomic. Waiting
// workgroups poll with device-scope loads and sleep between polls; each counter and flag sits in
// a 128-byte line of its own. The count role reads what other count workgroups wrote with
// device-scope loads; a send workgroup takes one device-scope acquire after its wait (thread 0,
// passed on by the workgroup barrier) and then reads the offsets with ordinary loads.
//
// Progress. A waiting workgroup only waits for count workgroups, and the host sizes the grid to
// what the device holds at once (the occupancy of this kernel times the compute units), so every
// workgroup it waits for is resident. Every wait is still bounded (opts.spin_ticks of the 100 MHz
// real-time clock): on expiry the workgroup records a give-up bit, stores nothing more of its
// role, and runs to its end. The last workgroup to finish writes the launch's status word (zero,
// or the give-up bits) and returns every synchronisation word to zero for the next call.
#include "layout_body.h"
#include "rows_body.h"

namespace epl {

constexpr int kSyncHist = 0 * kSyncStride;    // count workgroups done with their chunks
constexpr int kSyncScan = 1 * kSyncStride;    // count workgroups done with their scan items
constexpr int kSyncReady = 2 * kSyncStride;   // 1 once every offset the send role reads is published
constexpr int kSyncExit = 3 * kSyncStride;    // workgroups done
constexpr int kSyncStatus = 4 * kSyncStride;  // give-up bits of this launch
// Words of every line that the workgroups count at on their way to a counter above (workgroup_publish).
constexpr int kLeafHist = 8, kLeafExit = 16, kNoLeaf = 0;
constexpr int kGaveUpCount = 1;    // a count workgroup stopped waiting
constexpr int kGaveUpSend = 2;     // a send workgroup stopped waiting
constexpr int kGaveUpCombine = 4;  // a combine wave stopped waiting for a row
constexpr int kSentinelInX = 8;    // an input row held the sentinel

struct DecomposedArgs {
  FusedLayout F;               // what the row placement reads and writes
  int32_t* tok_nranks;         // K1 and K2 outputs and workspace
  int32_t* chunk_e;
  int32_t* chunk_r;
  int32_t* inval;
  uint32_t* fmask;
  int32_t* recv_cnt;
  int32_t* send_cnt;
  int32_t* rank_cnt;
  int32_t* seg_rel;
  int32_t* num_invalid;
  int32_t* cnt;                // [nblk][E] chunk-major expert counts
  const float* topk_w;         // the combine role (the layer variants): [T*k] weights
  u32x4* out;                  // [T][H] bf16
  uint64_t* marks;             // Token-Flag Fusion and Data-for-Checksum: [cap][cchunks] words, one per 1 KiB
  uint64_t epoch;              // this call's epoch: the flag value, or the checksum's salt
  int cchunks, crun;           // 1 KiB column chunks per row, and per combine task
  int batch;                   // tokens a send workgroup takes at a time, <= kWavesPerBlock
  const u32x4* x;
  u32x4* recv;
  int nv, pv;                  // x row and recv pitch in 16-byte vectors
  int64_t cap;
  int nc, ns;                  // count workgroups; workgroups that send (all, where the count workgroups join)
  int32_t* sync;               // [kSyncWords]
  int32_t* status;             // the call's wait status
  int64_t spin_ticks;
  int ready_target;
};

// Polls `word` with device-scope loads until it reaches `target` or `limit` ticks of the 100 MHz
// real-time clock pass. Every lane of the wave runs it with the same values.
// SLEEP: 64-cycle steps between polls.
template <int SLEEP>
__device__ __forceinline__ bool wait_at_least(int32_t* word, int target, int64_t limit) {
  const int64_t t0 = wall_clock64();
  while (ld32<true>(word) < target) {
    if (wall_clock64() - t0 > limit) return false;
    __builtin_amdgcn_s_sleep(SLEEP);
  }
  return true;
}

// The count workgroups wait for each other and poll often; the send workgroups, four times as many, wait
// for all of it, and their polls go to the memory channel that the counters sit in.
constexpr int kSleepCount = 2, kSleepReady = 8;

// The whole workgroup waits: thread 0 polls, the others park at the barrier. With ACQUIRE, thread
// 0 then takes a device-scope acquire (it invalidates the compute unit's L1 and the XCD's L2 of
// lines other XCDs may have changed), and the barrier passes it to the whole workgroup: its plain
// loads after the wait see everything published before the word was set.
template <bool ACQUIRE = false>
__device__ __forceinline__ bool workgroup_wait(int32_t* word, int target, int64_t limit, int32_t* flag) {
  if (threadIdx.x == 0) {
    const bool ok = wait_at_least<ACQUIRE ? kSleepReady : kSleepCount>(word, target, limit);
    if (ACQUIRE && ok) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *flag = ok ? 1 : 0;
  }
  __syncthreads();
  const bool ok = *flag != 0;
  __syncthreads();  // every thread has read the flag before it can be rewritten
  return ok;
}

// Counts workgroup i of n at the counter `root`, once the workgroup's own stores are complete; true in
// thread 0 of the last one. Adds to one address are served one after another, so where all workgroups
// arrive together they add to kLeaves words (word `leaf` of each synchronisation line) and the last of
// each leaf adds to the root: the counts of 256 workgroups meet 3-4 us after the last has finished, 6-7
// with one counter. Few workgroups, and all with kNoLeaf, add to the root (arrivals spread by more than an add
// takes: the second level would only cost its round trip; layout and dispatch of 32 tokens on 16 ranks 28.6 us with
// it, 25.9 without).
constexpr int kLeaves = kSyncWords / kSyncStride;
constexpr int kLeafFrom = 128;  // fewer workgroups add to the root
__device__ __forceinline__ int leaf_count(int n) { return n < kLeafFrom ? n : kLeaves; }
__device__ __forceinline__ bool workgroup_publish(int32_t* sync, int root, int leaf, int i, int n) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x != 0) return false;
  auto add = [&](int word) {
    return __hip_atomic_fetch_add(&sync[word], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (leaf == kNoLeaf || n < kLeafFrom) return add(root) == n - 1;
  const int l = i % kLeaves;
  if (add(l * kSyncStride + leaf) != (n - l + kLeaves - 1) / kLeaves - 1) return false;
  return add(root) == leaf_count(n) - 1;
}

__device__ __forceinline__ void count_role(const DecomposedArgs& A, int i, int32_t* lds, int32_t* red,
                                           int32_t* scratch, int32_t* seg_start, int32_t* flag) {
  const Geom& G = A.F.G;
  for (int b = i; b < G.nblk; b += A.nc) {
    hist_chunk<true>(G, b, A.F.idx, A.tok_nranks, A.chunk_e, A.chunk_r, A.inval, A.fmask, lds, red, A.cnt);
    __syncthreads();  // the next chunk reuses the LDS
  }
  workgroup_publish(A.sync, kSyncHist, kLeafHist, i, A.nc);
  if (!workgroup_wait(&A.sync[kSyncHist], leaf_count(A.nc), A.spin_ticks, flag) && threadIdx.x == 0)
    atomicOr(&A.sync[kSyncStatus], kGaveUpCount);
  for (int item = i; item < G.E + G.R + 1; item += A.nc) {
    scan_item<true>(G, item, A.chunk_e, A.chunk_r, A.inval, A.recv_cnt, A.send_cnt, A.rank_cnt, A.seg_rel,
                    A.num_invalid, scratch, seg_start, A.cnt);
    __syncthreads();
  }
  if (workgroup_publish(A.sync, kSyncScan, kNoLeaf, i, A.nc)) {
    // Every count workgroup's stores completed before its count; publish the offsets.
    __hip_atomic_store(&A.sync[kSyncReady], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // expert_off, rank_off and one slice of seg_off, from the published totals.
  if (workgroup_wait(&A.sync[kSyncReady], 1, A.spin_ticks, flag)) {
    offsets_block(A.F, i, A.nc, lds);
  } else {
    if (threadIdx.x == 0) atomicOr(&A.sync[kSyncStatus], kGaveUpCount);
  }
}

// ------------------------------------------------------------------------ Sentinel Polling
// In the layer variant the workgroups go on to gather the dispatched rows (identity experts:
// the combine reads the receive buffer itself) while the send workgroups are still writing them,
// with no barrier in between: the paper's Sentinel Polling (Data-as-Flag). Every receive row holds
// the reserved bf16 pattern EPL_SENTINEL_BF16 (a negative NaN with every payload bit set, which
// arithmetic does not produce) in every element before the send role writes it. A combine lane
// loads its 16 bytes of a row with device-scope loads until none of its 8 elements is the
// sentinel. MI355X gives no 512-byte store atomicity, so the check is per element rather than on
// a leading flag field: a row counts as arrived, for one lane, exactly when each of that lane's
// elements has been written, whatever the order or granularity of the stores. After folding a
// row the lane writes the sentinel back over what it read, so the buffer is ready for the next
// layer (the paper's reset after consumption). The send role checks every input vector for the
// sentinel and reports one (a row that carries it would never count as arrived).
constexpr uint32_t kSentinelPair = 0xFFFFFFFFu;  // two bf16 sentinels

__device__ __forceinline__ bool holds_sentinel(u32x4 v) {
  bool any = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) any |= ((v[i] & 0xFFFFu) == 0xFFFFu) | ((v[i] >> 16) == 0xFFFFu);
  return any;
}

// ------------------------------------------------------------------------ Token-Flag Fusion, Data-for-Checksum
// The paper's other two Data-as-Flag variants, for a GPU without multi-word store atomicity. Both
// keep one 64-bit word per (packed row, 1 KiB column chunk) in `marks`, beside the rows, and an
// epoch that the caller changes on every call, so nothing has to be reset between layers.
// * Token-Flag Fusion: the paper stores a flag field and the payload in one atomic 512-byte block.
//   Here a send wave waits until its own device-scope row stores are complete (vmcnt), then stores
//   the epoch into the marks of the chunks it wrote; a combine wave polls the mark until it holds
//   the epoch and only then loads the chunk. The wait on the sender is what the fused flag avoids
//   on the paper's fabric.
// * Data-for-Checksum: the paper's receiver waits for a checksum of the batch's leading markers,
//   written after the batch. Without block atomicity a marker does not vouch for the rest of its
//   block, so the checksum here covers every byte of its 1 KiB chunk: a 64-bit hash of the chunk,
//   salted with the epoch. The send wave stores it with no wait at all; a combine wave loads the
//   chunk and the mark and accepts the chunk when the hash of what it loaded, salted the same way,
//   equals the mark (else it loads both again). Stale data, a stale mark, or a chunk only partly
//   written all fail the comparison except with probability about 2^-64.
__device__ __forceinline__ uint64_t ld64_dev(const uint64_t* p) {
  return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st64_dev(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The SplitMix64 output function (Steele, Lea and Flood, "Fast splittable pseudorandom number
// generators", OOPSLA 2014): a bijective 64-bit mixer.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// One lane's 16 bytes at lane position `lane` of its chunk, mixed; lanes outside the row give 0.
__device__ __forceinline__ uint64_t lane_hash(u32x4 v, bool on, int lane) {
  const uint64_t a = (uint64_t)v[0] | ((uint64_t)v[1] << 32);
  const uint64_t b = (uint64_t)v[2] | ((uint64_t)v[3] << 32);
  return on ? mix64(a ^ mix64(b + 0x9E3779B97F4A7C15ull * (uint64_t)(lane + 1))) : 0;
}

// XOR over the wave's 64 lanes; every lane returns the total.
__device__ __forceinline__ uint64_t wave_xor64(uint64_t h) {
  int lo = (int)(uint32_t)h, hi = (int)(uint32_t)(h >> 32);
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) {
    lo ^= __shfl_xor(lo, m, kWave);
    hi ^= __shfl_xor(hi, m, kWave);
  }
  return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

__device__ __forceinline__ uint64_t epoch_salt(uint64_t epoch) { return mix64(epoch ^ 0x5851F42D4C957F2Dull); }

// The wave's index in its workgroup; the compiler does not see by itself that it is the same in all lanes.
template <int SYNC, int FORM>
__device__ __forceinline__ int wave_index() {
  const int w = threadIdx.x / kWave;
  return scalar_wave(FORM, SYNC != kDafNone) ? __builtin_amdgcn_readfirstlane(w) : w;
}

// Sends the batches j, j + ns, ... of A.batch consecutive tokens, after waiting for the offsets once
// the first loads are issued. One wave places each token of the batch (its rows go to the others
// through LDS), then the four waves take the batch's (token, 1 KiB column chunk) units in turn. A token
// is placed once, and rows are written in the 1 KiB pieces that spread best over the memory. A wave
// loads AHEAD units together (send_ahead). Returns false if it gave up.
// Against one 4 KiB unit per wave at a time, each with a placement of its own, whole layer: 16 ranks x
// 128 tokens x 2048 columns 49.0 -> 44.9 us, 32 x 64 x 7168 113.0 -> 107.8, 64 x 128 x 7168 411 -> 408; with the
// next unit's load in flight under the stores 51, 125 and 410.
// Measured against handing out batches of units from a launch-wide counter, with the count
// workgroups joining once their counting was done: that was slower (decode 416.7 against
// 396.8 us per layer, the Qwen3-30B shape 61.2 against 50.7 us), the counter's atomics serialising.
template <int SYNC, int FORM>
__device__ __forceinline__ bool send_role(const DecomposedArgs& A, int j, int32_t* lds, int32_t* flag) {
  const int lane = threadIdx.x % kWave;
  constexpr int AHEAD = send_ahead(FORM, SYNC != kDafNone);
  const int w = wave_index<SYNC, FORM>();
  const int k = A.F.G.k;
  const int nv = A.nv;
  int32_t* rows_lds = lds;  // [kWavesPerBlock][k]
  int32_t* hist = lds + kWavesPerBlock * EPL_MAX_TOPK + w * (A.F.G.E + A.F.G.R);
  const uint64_t salt = epoch_salt(A.epoch);
  bool waited = false;
  // The loop bounds are the workgroup's, so every wave reaches the same barriers.
  for (int64_t g0 = (int64_t)j * A.batch; g0 < A.F.G.T; g0 += (int64_t)A.ns * A.batch) {
    const int ntok = (int)std::min<int64_t>(A.batch, A.F.G.T - g0);  // <= kWavesPerBlock
    const int units = ntok * A.cchunks;
    u32x4 buf[AHEAD];
    auto load_units = [&](int u0) {  // units u0, u0 + 4, ... of this wave; past the last an empty resource, not a branch
#pragma unroll
      for (int q = 0; q < AHEAD; ++q) {
        const int u = min(u0 + q * kWavesPerBlock, units - 1);
        const int tl = u / A.cchunks;
        const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<u32x4*>(A.x + (g0 + tl) * nv), 0, u0 + q * kWavesPerBlock < units ? nv * 16 : 0, kBufferRsrcWord3);
        buf[q] = __builtin_amdgcn_raw_buffer_load_b128(xs, ((u - tl * A.cchunks) * kWave + lane) * 16, 0, 0);
      }
    };
    load_units(w);
    if (!waited) {
      waited = true;
      if (!workgroup_wait<true>(&A.sync[kSyncReady], A.ready_target, A.spin_ticks, flag)) {
        if (threadIdx.x == 0) atomicOr(&A.sync[kSyncStatus], kGaveUpSend);
        return false;  // uniform over the workgroup: nothing is stored
      }
    }
    if (w < ntok) {
      const int r = token_rows(A.F, g0 + w, true, hist, lane);
      if (lane < k) rows_lds[w * k + lane] = r;
    }
    __syncthreads();
    for (int u0 = w; u0 < units; u0 += AHEAD * kWavesPerBlock) {
      if (u0 != w) load_units(u0);
#pragma unroll
      for (int q = 0; q < AHEAD; ++q) {
        const int u = u0 + q * kWavesPerBlock;
        if (u >= units) break;
        const int tl = u / A.cchunks;
        const int c = u - tl * A.cchunks;
        const int v = c * kWave + lane;
        const int my_row = lane < k ? rows_lds[tl * k + lane] : -1;
        if constexpr (SYNC == kDafSentinel) {
          if (__ballot(v < nv && holds_sentinel(buf[q])) != 0 && lane == 0)
            atomicOr(&A.sync[kSyncStatus], kSentinelInX);
        }
        for (int jj = 0; jj < k; ++jj) {
          const int row = __builtin_amdgcn_readlane(my_row, jj);
          if (row < 0 || row >= A.cap) continue;
          if (v < nv) store_row_policy<kCachePolicySc1>(buf[q], A.recv + (int64_t)row * A.pv, nv, v);
        }
        if constexpr (SYNC == kDafChecksum) {
          const uint64_t m = wave_xor64(lane_hash(buf[q], v < nv, lane)) ^ salt;
          if (my_row >= 0 && my_row < A.cap) st64_dev(&A.marks[(int64_t)my_row * A.cchunks + c], m);
        }
      }
    }
    if constexpr (SYNC == kDafFlag) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's device-scope row stores are complete
      for (int u = w; u < units; u += kWavesPerBlock) {
        const int tl = u / A.cchunks;
        const int my_row = lane < k ? rows_lds[tl * k + lane] : -1;
        if (my_row >= 0 && my_row < A.cap) st64_dev(&A.marks[(int64_t)my_row * A.cchunks + u - tl * A.cchunks], A.epoch);
      }
    }
    __syncthreads();  // every wave has read the rows before the next batch rewrites them
  }
  return true;
}

// Loads vector v of packed row `row` (nothing, and zeros, for row < 0: its resource is empty).
__device__ __forceinline__ u32x4 gather_vec(const u32x4* y, int row, int pv, int nv, int v) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4*>(y + (int64_t)max(row, 0) * pv), 0,
                                                                     row >= 0 ? nv * 16 : 0, kBufferRsrcWord3);
  return __builtin_amdgcn_raw_buffer_load_b128(r, v * 16, 0, kCachePolicySc1);
}

// Combine tasks (token g, a run of 1 KiB column chunks): one wave per task, waves iterating on their
// own. Each wave works out its token's rows as the send role does (no metadata written), then for
// each chunk gathers the valid rows and folds them in j order, acc = fmaf(w_j, y_j, acc) from +0,
// bf16 round-to-nearest-even, as the combine kernel does.
//
// What bounds it is latency: a row's load is a round trip to memory (device-scope, past the L2), and
// placing a token costs about as much again. So all of a chunk's rows (up to kAhead at a time; two with few
// choices, where the other six would be empty loads and checks) are
// loaded before any is checked, a wave keeps its token for as many chunks as leave every wave a task, and
// every workgroup of the launch combines. Against combine workgroups of their own that loaded one row after
// another, whole layer: 16 ranks x 128 tokens x 2048 columns sentinel 68.9 -> 55.1 us, flag 75.4 -> 46.5,
// checksum 75.4 -> 60.0; 32 x 64 x 7168 sentinel 192 -> 156; 64 x 128 x 7168 967 -> 630.
template <int SYNC, int FORM>
__device__ __forceinline__ void combine_role(const DecomposedArgs& A, int ci, int32_t* lds) {
  constexpr int kAhead = FORM == kFormFew ? kFewChoices : 8;
  const Geom& G = A.F.G;
  const int lane = threadIdx.x % kWave;
  const int w = wave_index<SYNC, FORM>();
  const int k = G.k;
  int32_t* hist = lds + kWavesPerBlock * EPL_MAX_TOPK + w * (G.E + G.R);
  const int nv = A.nv;
  const int runs = (A.cchunks + A.crun - 1) / A.crun;  // per token
  const int64_t tasks = G.T * runs;
  const int64_t stride = (int64_t)gridDim.x * kWavesPerBlock;
  const u32x4* y = A.recv;
  const uint64_t salt = epoch_salt(A.epoch);
  bool arrived = true;
  for (int64_t u = (int64_t)ci * kWavesPerBlock + w; u < tasks && arrived; u += stride) {
    const int64_t g = u / runs;
    const int c0 = (int)(u - g * runs) * A.crun;
    const int c1 = min(c0 + A.crun, A.cchunks);
    const int wbits = __builtin_bit_cast(int, A.topk_w[g * k + min(lane, k - 1)]);
    const int rows = token_rows(A.F, g, false, hist, lane);
    int c = c0;
    for (; c < c1; ++c) {
      const int v = c * kWave + lane;
      const bool on = v < nv;
      const int vl = min(v, nv - 1);
      // Lane j's mark of this chunk (Token-Flag Fusion, Data-for-Checksum).
      const uint64_t* mark = A.marks + (int64_t)max(rows, 0) * A.cchunks + c;
      if constexpr (SYNC == kDafFlag) {  // every row's chunk is there before any is loaded
        int64_t t0 = -1;
        while (__ballot(rows >= 0 && ld64_dev(mark) != A.epoch) != 0) {
          if (t0 < 0) t0 = wall_clock64();
          if (wall_clock64() - t0 > A.spin_ticks) {
            arrived = false;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
        if (!arrived) break;  // wave-uniform, as is every exit below
      }
      float acc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
      for (int j0 = 0; j0 < k && arrived; j0 += kAhead) {
        u32x4 buf[kAhead];
        int row[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
          row[q] = __builtin_amdgcn_readlane(rows, j0 + q);  // -1 in the lanes past k (k <= 32)
          buf[q] = gather_vec(y, row[q], A.pv, nv, vl);
        }
        if constexpr (SYNC != kDafFlag) {
          auto load_mark = [&] { return SYNC == kDafChecksum && rows >= 0 ? ld64_dev(mark) : 0; };
          uint64_t m = load_mark();
          // Whether every lane's part of choice jj's chunk, loaded as val, has arrived.
          auto is_there = [&](u32x4 val, int jj) {
            if constexpr (SYNC == kDafChecksum) {
              const uint64_t mj = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m, jj) |
                                  (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(m >> 32), jj) << 32;
              return __ballot((wave_xor64(lane_hash(val, on, lane)) ^ salt) != mj) == 0;
            }
            return __ballot(holds_sentinel(val)) == 0;
          };
          int64_t t0 = -1;
          while (true) {
            uint32_t missing = 0;  // bit q: choice j0 + q has not arrived
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
              if (row[q] >= 0 && !is_there(buf[q], j0 + q)) missing |= 1u << q;
            if (missing == 0) break;
            // Poll one missing row until it is there (eight polled at once slow the sends down), then
            // load all that were missing again (keeping the polled value costs registers and was no faster).
            const int jp = j0 + __builtin_ctz(missing);
            const int rp = __builtin_amdgcn_readlane(rows, jp);
            if (t0 < 0) t0 = wall_clock64();
            do {
              if (wall_clock64() - t0 > A.spin_ticks) {
                arrived = false;
                break;
              }
              __builtin_amdgcn_s_sleep(4);
              m = load_mark();
            } while (!is_there(gather_vec(y, rp, A.pv, nv, vl), jp));
            if (!arrived) break;
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
              if ((missing >> q) & 1u) buf[q] = gather_vec(y, row[q], A.pv, nv, vl);
            m = load_mark();
          }
          if (!arrived) break;
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
          if (row[q] < 0) continue;
          const float wj = __builtin_bit_cast(float, __builtin_amdgcn_readlane(wbits, j0 + q));
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc[2 * i] = fmaf(wj, bf16lo_to_f32(buf[q][i]), acc[2 * i]);
            acc[2 * i + 1] = fmaf(wj, bf16hi_to_f32(buf[q][i]), acc[2 * i + 1]);
          }
        }
      }
      if (!arrived) break;
      if (on) {
        u32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = f32x2_to_bf16x2(acc[2 * i], acc[2 * i + 1]);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(A.out + g * nv, 0, nv * 16, kBufferRsrcWord3);
        __builtin_amdgcn_raw_buffer_store_b128(o, r, v * 16, 0, kCachePolicySc1Nt);
      }
    }
    if constexpr (SYNC == kDafSentinel) {
      // What was consumed, back to the sentinel for the next layer: after the last chunk, as a load
      // issued behind stores would wait for them.
      const u32x4 s = {kSentinelPair, kSentinelPair, kSentinelPair, kSentinelPair};
      for (int cr = c0; cr < c; ++cr) {
        const int v = cr * kWave + lane;
        for (int j = 0; j < k; ++j) {
          const int row = __builtin_amdgcn_readlane(rows, j);
          if (row >= 0 && v < nv) store_row_policy<kCachePolicySc1>(s, A.recv + (int64_t)row * A.pv, nv, v);
        }
      }
    }
  }
  if (!arrived && lane == 0) atomicOr(&A.sync[kSyncStatus], kGaveUpCombine);
}

// The split form's combine: one (token, 1 KiB column chunk) per wave at a time, its rows one after another, each
// loaded until it is there and folded (and, for Sentinel Polling, reset) before the next. The task at hand is
// short, and so is the code (see send_ahead).
template <int SYNC>
__device__ __forceinline__ void combine_rows(const DecomposedArgs& A, int ci, int groups, int32_t* lds) {
  const Geom& G = A.F.G;
  const int lane = threadIdx.x % kWave;
  const int w = wave_index<SYNC, kFormSplit>();
  const int k = G.k;
  int32_t* hist = lds + kWavesPerBlock * EPL_MAX_TOPK + w * (G.E + G.R);
  const int nv = A.nv;
  const int64_t units = G.T * A.cchunks;
  const int64_t stride = (int64_t)groups * kWavesPerBlock;
  const u32x4* y = A.recv;
  const uint64_t salt = epoch_salt(A.epoch);
  for (int64_t u = (int64_t)ci * kWavesPerBlock + w; u < units; u += stride) {
    const int64_t g = u / A.cchunks;
    const int c = (int)(u - g * A.cchunks);
    const int rows = token_rows(A.F, g, false, hist, lane);
    const int v = c * kWave + lane;
    const bool on = v < nv;
    const int vl = min(v, nv - 1);
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
    for (int j = 0; j < k; ++j) {
      const int row = __builtin_amdgcn_readlane(rows, j);
      if (row < 0) continue;
      const float wj = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, A.topk_w[g * k + j])));
      const uint64_t* mark = A.marks + (int64_t)row * A.cchunks + c;
      u32x4 val;
      // Loads the lane's vector; whether the whole chunk of the row has arrived (wave-uniform).
      auto load = [&] {
        if constexpr (SYNC == kDafFlag) {
          if (ld64_dev(mark) != A.epoch) return false;
          val = gather_vec(y, row, A.pv, nv, vl);
          return true;
        } else if constexpr (SYNC == kDafChecksum) {
          const uint64_t m = ld64_dev(mark);
          val = gather_vec(y, row, A.pv, nv, vl);
          return (wave_xor64(lane_hash(val, on, lane)) ^ salt) == m;
        } else {
          val = gather_vec(y, row, A.pv, nv, vl);
          return __ballot(holds_sentinel(val)) == 0;
        }
      };
      if (!load()) {
        const int64_t t0 = wall_clock64();
        do {
          if (wall_clock64() - t0 > A.spin_ticks) {  // wave-uniform: stop, store nothing more
            if (lane == 0) atomicOr(&A.sync[kSyncStatus], kGaveUpCombine);
            return;
          }
          __builtin_amdgcn_s_sleep(1);
        } while (!load());
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[2 * i] = fmaf(wj, bf16lo_to_f32(val[i]), acc[2 * i]);
        acc[2 * i + 1] = fmaf(wj, bf16hi_to_f32(val[i]), acc[2 * i + 1]);
      }
      if (SYNC == kDafSentinel && on) {  // consumed: back to the sentinel for the next layer
        const u32x4 s = {kSentinelPair, kSentinelPair, kSentinelPair, kSentinelPair};
        store_row_policy<kCachePolicySc1>(s, A.recv + (int64_t)row * A.pv, nv, v);
      }
    }
    if (on) {
      u32x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = f32x2_to_bf16x2(acc[2 * i], acc[2 * i + 1]);
      const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(A.out + g * nv, 0, nv * 16, kBufferRsrcWord3);
      __builtin_amdgcn_raw_buffer_store_b128(o, r, v * 16, 0, kCachePolicySc1Nt);
    }
  }
}

// The last workgroup to finish writes the status word and zeroes the synchronisation words. Every
// other workgroup has passed all its waits by then.
__device__ __forceinline__ void finish(const DecomposedArgs& A) {
  if (workgroup_publish(A.sync, kSyncExit, kLeafExit, (int)blockIdx.x, (int)gridDim.x)) {
    st32<true>(A.status, ld32<true>(&A.sync[kSyncStatus]));
    for (int i = 0; i < kSyncWords; i += kLeafHist) st32<true>(&A.sync[i], 0);
  }
}

// Every workgroup of a layer variant goes on to combine when its own role is done: the whole device
// sends first, and by the time a workgroup combines, most of what it gathers has arrived. In the split form
// the workgroups past the senders combine meanwhile.
template <int SYNC, int FORM>
__global__ void __launch_bounds__(kLayoutThreads) __attribute__((amdgpu_waves_per_eu(5)))
    decomposed_kernel(DecomposedArgs A) {
  static_assert(kDispatchThreads == kLayoutThreads, "both roles run in 256-thread workgroups");
  static_assert(kWavesPerBlock == kSendBatch, "a send workgroup's waves place one token each");
  extern __shared__ int32_t lds[];
  __shared__ int32_t red[kLayoutWaves];
  __shared__ int32_t scratch[kLayoutWaves];
  __shared__ int32_t seg_start[EPL_MAX_EXPERTS + 1];
  __shared__ int32_t flag;
  bool ready = true;  // the offsets are published, and acquired
  bool sends = true;
  int j = (int)blockIdx.x - A.nc;
  if (j < 0) {
    count_role(A, (int)blockIdx.x, lds, red, scratch, seg_start, &flag);
    sends = A.ns > (int)gridDim.x - A.nc;
    j += (int)gridDim.x;  // after the send workgroups: gridDim - nc + i
    if (sends || (SYNC != kDafNone && FORM != kFormSplit))
      ready = workgroup_wait<true>(&A.sync[kSyncReady], A.ready_target, A.spin_ticks, &flag);
  }
  if constexpr (FORM == kFormSplit) {
    if (j >= A.ns) {  // also the count workgroups, whose j lies past the senders
      sends = false;
      if ((int)blockIdx.x >= A.nc) {
        if (workgroup_wait<true>(&A.sync[kSyncReady], A.ready_target, A.spin_ticks, &flag))
          combine_rows<SYNC>(A, j - A.ns, (int)gridDim.x - A.nc - A.ns, lds);
        else if (threadIdx.x == 0)
          atomicOr(&A.sync[kSyncStatus], kGaveUpCombine);
      }
    }
  }
  if (sends && ready) ready = send_role<SYNC, FORM>(A, j, lds, &flag);
  if constexpr (SYNC != kDafNone && FORM != kFormSplit) {
    if (ready)
      combine_role<SYNC, FORM>(A, (int)blockIdx.x, lds);
    else if (threadIdx.x == 0)
      atomicOr(&A.sync[kSyncStatus], kGaveUpCombine);
  }
  finish(A);
}

// ------------------------------------------------------------------------ host
namespace {

typedef void (*DecomposedKernel)(DecomposedArgs);
template <int SYNC>
DecomposedKernel kernel_of_form(int form) {
  if constexpr (SYNC != kDafNone) {
    if (form == kFormSplit) return decomposed_kernel<SYNC, kFormSplit>;
  } else {
    if (form == kFormWide) return decomposed_kernel<SYNC, kFormWide>;
  }
  return form == kFormFew ? decomposed_kernel<SYNC, kFormFew> : decomposed_kernel<SYNC, kFormGeneral>;
}

DecomposedKernel kernel_of(int sync, int form) {
  switch (sync) {
    case kDafSentinel: return kernel_of_form<kDafSentinel>(form);
    case kDafFlag: return kernel_of_form<kDafFlag>(form);
    case kDafChecksum: return kernel_of_form<kDafChecksum>(form);
    default: return kernel_of_form<kDafNone>(form);
  }
}

size_t decomposed_lds_bytes(const Geom& g) {
  const size_t hist = (size_t)g.E + g.R;                                        // K1
  const size_t rows = (size_t)kWavesPerBlock * (EPL_MAX_TOPK + g.E + g.R);      // row placement
  const size_t meta = (size_t)g.E + 1;                                           // offsets
  return sizeof(int32_t) * std::max(hist, std::max(rows, meta));
}

}  // namespace

hipError_t plan_decomposed(const Geom& g, int H, int count_groups, int sync, DecomposedPlan* plan) {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  for (int form = decomposed_form(g, H, sync);; form = joined_form(g, H, sync)) {
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel_of(sync, form), kLayoutThreads, decomposed_lds_bytes(g));
    if (e != hipSuccess) return e;
    *plan = split_decomposed(g, H, count_groups, sync, form, per_cu * cus, cus);
    // A count_groups that leaves room for a single workgroup: it has to send and to combine.
    if (form != kFormSplit || plan->grid <= plan->capacity) return hipSuccess;
  }
}

hipError_t launch_decomposed(const Geom& g, const int32_t* idx, int32_t* ws, const epl_layout_buffers& L,
                             const void* x, void* recv, int H, int pitch, int64_t cap, const DecomposedOpts& opts,
                             int32_t* wait_status, hipStream_t stream, int sync, const float* topk_w, void* out,
                             uint64_t* marks, uint64_t epoch) {
  DecomposedPlan plan;
  hipError_t e = plan_decomposed(g, H, opts.count_groups, sync, &plan);
  if (e != hipSuccess) return e;
  if (plan.grid > plan.capacity) return hipErrorLaunchOutOfResources;  // refused on the host before this
  const WsLayout wl = ws_layout(g);
  DecomposedArgs A;
  A.F = FusedLayout{g,          idx,          ws + wl.chunk_e, ws + wl.chunk_r,
                    ws + wl.recv_cnt, ws + wl.seg_rel, reinterpret_cast<const uint32_t*>(ws + wl.fmask),
                    L.expert_off, L.rank_off,     L.seg_off,       L.pair_row,
                    L.pair_rslot, L.recv_src,     L.recv_j};
  A.tok_nranks = L.tok_nranks;
  A.chunk_e = ws + wl.chunk_e;
  A.chunk_r = ws + wl.chunk_r;
  A.inval = ws + wl.inval;
  A.fmask = reinterpret_cast<uint32_t*>(ws + wl.fmask);
  A.recv_cnt = ws + wl.recv_cnt;
  A.send_cnt = L.send_cnt;
  A.rank_cnt = L.rank_cnt;
  A.seg_rel = ws + wl.seg_rel;
  A.num_invalid = L.num_invalid;
  A.cnt = ws + wl.cnt;
  A.topk_w = topk_w;
  A.out = static_cast<u32x4*>(out);
  A.marks = marks;
  A.epoch = epoch;
  A.x = static_cast<const u32x4*>(x);
  A.recv = static_cast<u32x4*>(recv);
  A.nv = H / 8;
  A.pv = pitch / 8;
  A.cchunks = (A.nv + kWave - 1) / kWave;
  A.cap = cap;
  A.nc = plan.count_groups;
  A.ns = plan.senders;
  A.crun = plan.combine_run;
  A.batch = plan.batch;
  A.sync = ws + wl.sync;
  A.status = wait_status;
  A.spin_ticks = opts.spin_ticks;
  A.ready_target = opts.ready_target;
  const size_t lds = decomposed_lds_bytes(g);
  hipLaunchKernelGGL(kernel_of(sync, plan.form), dim3(plan.grid), dim3(kLayoutThreads), lds, stream, A);
  return hipGetLastError();
}

// The fill kernel: every 16-byte vector of the buffer set to sentinels.
__global__ void sentinel_fill_kernel(u32x4* __restrict__ buf, int64_t nvec) {
  const u32x4 s = {kSentinelPair, kSentinelPair, kSentinelPair, kSentinelPair};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * blockDim.x)
    buf[i] = s;
}

hipError_t launch_sentinel_fill(void* buf, int64_t nvec, hipStream_t stream) {
  if (nvec == 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((nvec + 255) / 256, 8192);
  hipLaunchKernelGGL(sentinel_fill_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, static_cast<u32x4*>(buf),
                     nvec);
  return hipGetLastError();
}

}  // namespace epl
