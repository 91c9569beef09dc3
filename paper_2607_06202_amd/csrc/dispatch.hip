// MoE dispatch on one GPU: write each token's row into the packed receive row of every valid
// (token, expert) pair.
//
// This is the paper's Token-Sending into pre-partitioned receive space (Implementation, global
// load/store; Background phase 2). Token-Reordering is fused in: the layout has already fixed
// every row, so each copy lands in its final slot.
//
// Work is cut into equal units, each a (token, column chunk) pair, one unit per wave. Every unit
// moves at most k copies of the same number of bytes, so the units are as balanced as the
// paper's equal token slices (Hierarchical Token-level Scheduling). Fine units also keep the
// last partial round of waves short. The token's chunk is read once with 16-byte loads and
// written k times with 16-byte stores.
//
// The fp8 variant quantises while copying. For each 128-element block the scale is
// s = max|x| / 448, and each element is stored as q = E4M3(x / s), RNE and saturating. It
// writes the same q row and scale row to all k destinations.
#include "rows_body.h"

namespace epl {

// The plain bf16 kernel: one (token, 1 KiB column chunk) per wave, two waves per workgroup, held at 4
// waves per SIMD. What bounds it is how scattered writes spread over the memory: in a write-only probe
// 14 KiB rows in random order take 5.3 TB/s in 4 KiB pieces and 5.56 in 1 KiB pieces (in sequential
// order 7.3). Small pieces of a row written from several XCDs (consecutive workgroups run on different
// ones) measured best, and few at a time. Whole layer, expert outputs in a buffer of their own, us for
// (piece, waves per workgroup, waves per SIMD):
// * EP=64 decode: 4 KiB, 4, any 397; 1 KiB, 4, any 396; 1 KiB, 4, 3 381; 1 KiB, 2, 3 / 4 / 5 / 6
//   379.4 / 378.8 / 381.4 / 390; 1 KiB, 7, 3 388; 1 KiB, 1, 4 379.4; 2 KiB, 2, 3 388; 4 KiB, 4, 3 399;
// * EP=256: 4 KiB, 4, 6 769; 1 KiB, 4, any 777; 1 KiB, 2, 2 / 3 / 4 / 5 785 / 743.4 / 742.6 / 750;
//   2 KiB, 2, 3 762; 4 KiB, 4, 3 785; neighbouring pieces on one XCD 773;
// * EP=32 prefill: 4 KiB, 4, 6 6112; 1 KiB, 2, 3 / 4 / 5 5873 / 5877 / 6041.
// Pieces of 512 or 256 bytes (several tokens per wave) were no faster (380-395 at decode). Loads of x
// with the nt policy cost 6 us at decode; buffer loads change nothing.
// With one or two choices a wave has little to write and more of them are needed: 6 waves per SIMD.
// Whole layer, 4 KiB pieces / 1 KiB at 4 / at 6 waves: top-1 of 32K rows of 7168 columns 456 / 459 / 433,
// of 64K rows of 1024 138.7 / 143.3 / 136.3; top-2 of 32K rows of 7168 606 / 575 / 585, of 32K rows of
// 512 55.1 / 57.2 / 55.5; top-4 of 16K rows of 4096 259 / 243 / 248.
constexpr int plain_waves_per_simd(bool few) { return few ? 6 : 4; }
template <bool FEW>
__global__ void __launch_bounds__(kPlainThreads)
    __attribute__((amdgpu_waves_per_eu(plain_waves_per_simd(FEW), plain_waves_per_simd(FEW))))
    dispatch_bf16_kernel(const u32x4* __restrict__ x, const int32_t* __restrict__ pair_row, u32x4* __restrict__ recv,
                         int64_t T, int k, int nv, int pv, int chunks, int64_t cap) {
  const int lane = threadIdx.x % kWave;
  const int64_t units = T * chunks;
  const int64_t stride = (int64_t)gridDim.x * kPlainWaves;
  for (int64_t u = (int64_t)blockIdx.x * kPlainWaves + threadIdx.x / kWave; u < units; u += stride) {
    const int64_t g = u / chunks;
    dispatch_bf16_unit(x, [&] { return lane < k ? pair_row[g * k + lane] : -1; }, recv, g, (int)(u - g * chunks), k, nv,
                       pv, cap, lane);
  }
}

// The fp8 kernel is capped at kFp8WavesPerSimd waves per SIMD. The compiler enforces the cap by
// reserving a larger register budget. Each wave writes up to k scattered 1 KiB q rows per 2 KiB of
// input, so fewer resident waves keep fewer concurrent random writes in flight; too few leave the
// per-element IEEE divisions of the quantiser exposed. Skewed fp8 EP=64, layout -> dispatch ->
// combine with the input rotated, dispatch per call over three alternating runs each:
// * 2 waves: 239.2-239.6 us;
// * 3 waves: 209.2-209.7 us;
// * 4 waves: 220.7-221.3 us;
// * 6 waves: 222.6-223.4 us;
// * 8 waves (uncapped): 222.6-222.8 us.
// With 2 waves, multiplying by a reciprocal instead of dividing (not the defined rounding) also
// brought it to 221 us, which places the 2-wave loss in the division latency.
constexpr int kFp8WavesPerSimd = 3;
__global__ void __launch_bounds__(kFp8Threads) __attribute__((amdgpu_waves_per_eu(kFp8WavesPerSimd, kFp8WavesPerSimd)))
    dispatch_fp8_kernel(const u32x4* __restrict__ x, const int32_t* __restrict__ pair_row, u32x4* __restrict__ recv,
                        float* __restrict__ recv_scale, int64_t T, int k, int H, int pq, int npass, int64_t cap) {
  const int lane = threadIdx.x % kWave;
  const int64_t units = T * npass;
  const int64_t stride = (int64_t)gridDim.x * kFp8Waves;
  for (int64_t u = (int64_t)blockIdx.x * kFp8Waves + threadIdx.x / kWave; u < units; u += stride) {
    const int64_t g = u / npass;
    dispatch_fp8_unit(x, [&] { return lane < k ? pair_row[g * k + lane] : -1; }, recv, recv_scale, g,
                      (int)(u - g * npass), k, H, pq, cap, lane);
  }
}

hipError_t launch_dispatch_bf16(const void* x, const int32_t* pair_row, void* recv, int64_t T, int k, int H,
                                int pitch, int64_t cap, hipStream_t stream) {
  if (T == 0) return hipSuccess;
  const int nv = H / 8;
  const int chunks = (nv + kWave - 1) / kWave;
  const int64_t units = T * chunks;
  const dim3 grid(unit_grid(units, kPlainWaves, kPlainThreads));
  const u32x4* xv = static_cast<const u32x4*>(x);
  u32x4* rv = static_cast<u32x4*>(recv);
  if (k <= kFewChoices)
    hipLaunchKernelGGL(dispatch_bf16_kernel<true>, grid, dim3(kPlainThreads), 0, stream, xv, pair_row, rv, T, k, nv,
                       pitch / 8, chunks, cap);
  else
    hipLaunchKernelGGL(dispatch_bf16_kernel<false>, grid, dim3(kPlainThreads), 0, stream, xv, pair_row, rv, T, k, nv,
                       pitch / 8, chunks, cap);
  return hipGetLastError();
}

bool token_rows_ok(const Geom& g) {
  return g.CT * g.k <= kFusedSlots * kWave && g.E <= kFusedPer * kWave;
}

hipError_t launch_dispatch_fp8(const void* x, const int32_t* pair_row, void* recv, float* recv_scale, int64_t T,
                               int k, int H, int pitch, int64_t cap, hipStream_t stream) {
  if (T == 0) return hipSuccess;
  const int npass = (H + 1023) / 1024;
  const int64_t units = T * npass;
  const dim3 grid(unit_grid(units, kFp8Waves, kFp8Threads));
  hipLaunchKernelGGL(dispatch_fp8_kernel, grid, dim3(kFp8Threads), 0, stream, static_cast<const u32x4*>(x),
                     pair_row, static_cast<u32x4*>(recv), recv_scale, T, k, H, pitch / 16, npass, cap);
  return hipGetLastError();
}

// ------------------------------------------------------------------------ diagnostics
__global__ void debug_e4m3_kernel(const float* __restrict__ in, uint8_t* __restrict__ out, int64_t n) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= n) return;
  float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int t = 0; t < 4 && i + t < n; ++t) v[t] = in[i + t];
  const uint32_t q = f32x4_to_e4m3x4(v[0], v[1], v[2], v[3]);
  for (int t = 0; t < 4 && i + t < n; ++t) out[i + t] = (uint8_t)(q >> (8 * t));
}

hipError_t launch_debug_e4m3(const float* in, uint8_t* out, int64_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const int64_t threads = (n + 3) / 4;
  hipLaunchKernelGGL(debug_e4m3_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream, in, out, n);
  return hipGetLastError();
}

}  // namespace epl
