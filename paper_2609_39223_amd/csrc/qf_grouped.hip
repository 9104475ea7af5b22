// Device-side tables for the grouped (mixture-of-experts) layer: per-expert tile prefixes and
// expert orders, computed from the device row offsets so the host never reads them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qf_internal.h"

namespace qf {
namespace {

// Rounds of tiles on 8 XCDs of cus_xcd compute units, each of which takes an eighth of the tiles.
__device__ __forceinline__ int rounds_of(int tiles, int cols, int cus_xcd) {
  const int per = (tiles * cols + 7) / 8;
  return (per + cus_xcd - 1) / cus_xcd;
}

// tile_rows 0: row tiles of 128, or of 256 where the launch that reads tile_start (cols tile columns)
// takes less time in them.  A round of 128-row tiles takes 0.78 of one of 256-row tiles (8 experts,
// one round: forward 86 / 75 us, 35 of them the quantizer's), so what counts is how many rounds the
// rows' distribution makes of either.  Forward of a layer in 256- / 128-row tiles, us: 1 / 2 rounds
// (32 experts x 32 rows, 2048 x 2048, MXFP4) 165 / 188, 2 / 2 (x 48 rows) 203 / 187, 2 / 3 (64 x 16)
// 316 / 342, 3 / 3 (64 x 32) 358 / 339, 6 / 7 (128 x 16, 3072 x 2048) 931 / 903.
// One workgroup, a lane per expert; what it costs is latency (64 experts: 3 us less than with the
// sums and row counts walked by single lanes).
__global__ __launch_bounds__(1024) void grouped_prep_kernel(const int64_t* __restrict__ off, int E,
                                                            int tile_rows, int cols, int cus_xcd,
                                                            int* tile_start, int* order,
                                                            int* kstart) {
  __shared__ int64_t all_rows[1024];
  __shared__ int part[3][16];
  const int e = threadIdx.x, lane = e & 63, wv = e >> 6, nw = blockDim.x >> 6;
  const int64_t rows = e < E ? off[e + 1] - off[e] : 0;
  all_rows[e] = rows;
  // prefix sums over the experts of their 128-, 256- and 64-row units (the last: padded k ranges of dW)
  const int own[3] = {(int)((rows + 127) / 128), (int)((rows + 255) / 256), (int)((rows + 63) / 64)};
  int sum[3] = {own[0], own[1], own[2]}, tot[3] = {0, 0, 0};
#pragma unroll
  for (int d = 1; d < 64; d *= 2)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int t = __shfl_up(sum[q], d, 64);
      if (lane >= d) sum[q] += t;
    }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (lane == 63) part[q][wv] = sum[q];
    sum[q] -= own[q];
  }
  __syncthreads();
  for (int i = 0; i < nw; ++i)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      if (i == wv) sum[q] += tot[q];
      tot[q] += part[q][i];
    }
  if (tile_rows == 0)
    tile_rows = 7 * rounds_of(tot[0], cols, cus_xcd) <= 9 * rounds_of(tot[1], cols, cus_xcd) ? 128 : 256;
  if (e < E) tile_start[e] = tile_rows == 128 ? sum[0] : sum[1];
  if (e < E && kstart) kstart[e] = sum[2];
  if (e == 0) {
    tile_start[E] = tile_rows == 128 ? tot[0] : tot[1];
    tile_start[E + 1] = tile_rows;
    if (kstart) kstart[E] = tot[2];
  }
  if (e < E && order) {
    int rank = 0;
    for (int i = 0; i < E; ++i) {
      const int64_t ri = all_rows[i];
      rank += (ri > rows) || (ri == rows && i < e);
    }
    order[rank] = e;
  }
}

}  // namespace

hipError_t launch_grouped_prep(const int64_t* off, int64_t E, int tile_rows, int64_t N, int* tile_start,
                               int* order, int* kstart, hipStream_t s) {
  const int64_t cus = compute_units() / 8;
  hipLaunchKernelGGL(grouped_prep_kernel, dim3(1), dim3((unsigned)((E + 63) / 64 * 64)), 0, s, off,
                     (int)E, tile_rows, (int)((N + 255) / 256), (int)(cus < 1 ? 1 : cus), tile_start,
                     order, kstart);
  return hipGetLastError();
}

}  // namespace qf
