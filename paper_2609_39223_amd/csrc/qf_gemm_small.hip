// NT BF16 MFMA GEMM for gfx950 on outputs too small to fill the chip with the main kernel's tiles
// (qf_gemm_nt.hip): C[m, n] = sum_k A[m, k] B[n, k], both operands k-contiguous.
//
// What bounds these shapes is how fast one compute unit can copy operands into its LDS: about 52 GB/s
// of cold operands, whatever the tile and however many stages are in flight (256 x 256 tiles: a
// 64 KB stage per 1.25 us on 32 units as on 128).  So the work has to be spread over all units,
// and what counts is the operand bytes of the busiest one: gemm_tile picks the tile with the
// smallest ceil(tiles / units) (rows + columns).  Times of one product (operands rotating through
// 400 MB, us), the main kernel's 256 x 256 tiles against the tile picked here:
//     256 x   512 x  512   14.9 ->  3.4 (16 x 16)       512 x 4096 x 4096   85.7 -> 31.1 (128 x 64)
//      32 x  4096 x 4096   80.2 -> 11.8 (16 x 16)      1024 x 4096 x 4096   84.7 -> 41.7 (128 x 128)
//     256 x  4096 x 4096   83.3 -> 21.9 (64 x 64)      2048 x 1024 x 4096   83.0 -> 30.7 (128 x 64)
// Stages, LDS layout and swizzle, and the order in which every output element's products are
// summed (rising k, 32 at a time) are the main kernel's with norot.  Stages are handled in groups
// of U, NS groups of LDS buffers: while a step multiplies group s from registers, group s + 1's
// fragments are read and up to NS - 2 groups are under way (two-stage groups took 32 x 32 tiles
// from 0.22 to 0.20 us a stage where one wavefront per SIMD has nothing else to issue).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "qf_gemm_common.h"

namespace qf {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// s_waitcnt immediate: at most n vector memory operations outstanding, the rest not waited for
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// WM x WN wavefronts, each owning TM x TN accumulator blocks of 16 x 16; NS stage buffers.
// HALVES: the sum is formed as (stages before split_stage) + (the rest), as the main kernel's split
// of an FP32 product with a workspace does.
template <bool C_F32, bool HALVES, int WM, int WN, int TM, int TN, int U, int NS>
__global__ __launch_bounds__(WM * WN * 64) void gemm_small_kernel(NtArgs p) {
  constexpr int NW = WM * WN, NT = NW * 64;
  constexpr int TBM = 16 * WM * TM, TBN = 16 * WN * TN;
  constexpr int kOpStage = TBM * kRow, kStage = (TBM + TBN) * kRow;
  constexpr int NL = (TBM + TBN) / 8 / NW;        // 1 KB loads per wavefront and stage
  static_assert((TBM + TBN) % (8 * NW) == 0 && TBM % 8 == 0, "whole loads");
  constexpr int kPitch16 = TBN * 2 + 16, kPitch32 = TBN * 4 + 16;
  constexpr int kEpi = TBM * (C_F32 ? kPitch32 : kPitch16);
  constexpr int kSmem = NS * U * kStage > kEpi ? NS * U * kStage : kEpi;
  __shared__ __attribute__((aligned(16))) char smem[kSmem];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / WN, wn = w % WN;
  int64_t m0, n0;
  tile_origin<TBM, TBN>(p, remap_xcd(blockIdx.x, gridDim.x), m0, n0);
  const int64_t m_end = p.M, n_end = p.N, K = p.K;

  // Load q of wavefront w covers rows 8 r .. 8 r + 7 of the stage (A's rows, then B's), r = w NL + q;
  // rows past the edge load the last valid one.
  const __amdgpu_buffer_rsrc_t rsa = make_rsrc(p.A + m0 * p.lda, ((m_end - m0 - 1) * p.lda + K) * 2);
  const __amdgpu_buffer_rsrc_t rsb = make_rsrc(p.B + n0 * p.ldb, ((n_end - n0 - 1) * p.ldb + K) * 2);
  uint32_t goff[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) {
    const int r = w * NL + q;
    const bool isb = r >= TBM / 8;               // uniform
    const int64_t row = (isb ? r * 8 - TBM : r * 8) + (lane >> 3);
    const int64_t lim = (isb ? n_end - n0 : m_end - m0) - 1;
    const int c = (lane & 7) ^ ((4 * (r & 1) + (lane >> 4)) & 7);
    goff[q] = (uint32_t)(((row < lim ? row : lim) * (isb ? p.ldb : p.lda) + c * 8) * 2);
  }
  auto issue = [&](int s, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int r = w * NL + q;
      dma16_buf(r >= TBM / 8 ? rsb : rsa, goff[q], (uint32_t)s * (uint32_t)kRow,
                smem + buf * kStage + r * 1024);
    }
  };
  // fragment offsets, as in the main kernel
  int foa[2], fob[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int c = 4 * x + (lane >> 4), sw = (lane >> 1) & 7;
    foa[x] = (wm * 16 * TM + (lane & 15)) * kRow + ((c ^ sw) << 4);
    fob[x] = kOpStage + (wn * 16 * TN + (lane & 15)) * kRow + ((c ^ sw) << 4);
  }
  f32x4_t acc[TM][TN], first[HALVES ? TM : 1][HALVES ? TN : 1];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      acc[i][j] = f32x4_t{};
      if (HALVES) first[i][j] = f32x4_t{};
    }
  // Fragments of the U stages of a group (S slices of 32), two sets: a step multiplies one while
  // it reads the next group's into the other.
  constexpr int S = 2 * U;
  bf16x8_t fa[2][S][TM], fb[2][S][TN];
  const int nst = (int)(K / BK), n = (nst + U - 1) / U;
  const int last_u = nst - (n - 1) * U;          // stages of the last group
  auto issue_group = [&](int s, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s < n - 1 || u < last_u) issue(s * U + u, buf * U + u);
  };
  auto read_group = [&](int buf, auto par) __attribute__((always_inline)) {
    constexpr int P = decltype(par)::value;
#pragma unroll
    for (int x = 0; x < S; ++x) {
      const char* st = smem + (buf * U + x / 2) * kStage;
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[P][x][i] = *reinterpret_cast<const bf16x8_t*>(st + foa[x & 1] + i * 2048);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[P][x][j] = *reinterpret_cast<const bf16x8_t*>(st + fob[x & 1] + j * 2048);
    }
  };
  auto mfma_slice = [&](int P, int x) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[P][x][j], fa[P][x][i], acc[i][j],
                                                            0, 0, 0);
  };
  // Group g has landed for every wavefront; the NS - 3 groups after it may still be in flight (near
  // the end, where fewer or smaller ones follow, everything is waited for).
  auto wait_group = [&](int g) __attribute__((always_inline)) {
    if (g + NS - 3 < n - 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 3) * U * NL));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  int buf = 0;                                   // buffer of group s
  // FULL: groups s + 1 and s + NS - 1 exist and the latter is a whole one.  The main loop's steps
  // are straight-line code: where the reads are conditional, the wait before the MFMAs is for the
  // next group's reads too.
  auto step = [&](int s, auto par, auto full) __attribute__((always_inline)) {
    constexpr int P = decltype(par)::value;
    constexpr bool FULL = decltype(full)::value;
    const int nxt = buf == NS - 1 ? 0 : buf + 1, prev = buf == 0 ? NS - 1 : buf - 1;
    if (FULL) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 3) * U * NL));
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      // every wavefront has multiplied group s - 1, so its buffer is free
#pragma unroll
      for (int u = 0; u < U; ++u) issue((s + NS - 1) * U + u, prev * U + u);
      read_group(nxt, std::integral_constant<int, P ^ 1>{});
      __builtin_amdgcn_sched_barrier(0);
    } else if (s + 1 < n) {
      wait_group(s + 1);
      if (s + NS - 1 < n) issue_group(s + NS - 1, prev);
      read_group(nxt, std::integral_constant<int, P ^ 1>{});
    }
#pragma unroll
    for (int x = 0; x < S; ++x) {
      if (HALVES && x % 2 == 0 && s * U + x / 2 == (int)p.split_stage) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            first[i][j] = acc[i][j];
            acc[i][j] = f32x4_t{};
          }
      }
      if (FULL || s < n - 1 || x / 2 < last_u) mfma_slice(P, x);
    }
    __builtin_amdgcn_sched_barrier(0);
    buf = nxt;
  };
  if (n > 0) {
    const int pre = n < NS - 1 ? n : NS - 1;
    for (int s = 0; s < pre; ++s) issue_group(s, s);
    wait_group(0);
    read_group(0, std::integral_constant<int, 0>{});
    const std::integral_constant<int, 0> even{};
    const std::integral_constant<int, 1> odd{};
    int s = 0;
    for (; s + NS < n - 1; s += 2) {
      step(s, even, std::true_type{});
      step(s + 1, odd, std::true_type{});
    }
    for (; s < n; s += 2) {
      step(s, even, std::false_type{});
      if (s + 1 < n) step(s + 1, odd, std::false_type{});
    }
  }
  const int krem = (int)(K % BK);
  if (krem > 0) {
    // partial last stage: masked loads through registers into buffer 0
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int r = w * NL + q;
      const int c = (lane & 7) ^ ((4 * (r & 1) + (lane >> 4)) & 7);
      uint4 v = make_uint4(0, 0, 0, 0);
      const char* g = r >= TBM / 8 ? reinterpret_cast<const char*>(p.B + n0 * p.ldb)
                                   : reinterpret_cast<const char*>(p.A + m0 * p.lda);
      if (c * 8 < krem) v = *reinterpret_cast<const uint4*>(g + (int64_t)nst * kRow + goff[q]);
      *reinterpret_cast<uint4*>(smem + r * 1024 + lane * 16) = v;
    }
    __syncthreads();
    read_group(0, std::integral_constant<int, 0>{});
    mfma_slice(0, 0);
    if (krem > 32) mfma_slice(0, 1);
  }

  // epilogue, as in the main kernel: lane l owns columns 4 (l / 16) .. +3 of row l % 16 of a block
  __syncthreads();
  char* Cp = reinterpret_cast<char*>(p.C);
  const int er = wm * 16 * TM + (lane & 15), ec = wn * 16 * TN + 4 * (lane >> 4);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const f32x4_t a = HALVES ? first[i][j] + acc[i][j] : acc[i][j];
      if (C_F32)
        *reinterpret_cast<float4*>(smem + (er + 16 * i) * kPitch32 + (ec + 16 * j) * 4) =
            make_float4(a[0], a[1], a[2], a[3]);
      else
        *reinterpret_cast<uint2*>(smem + (er + 16 * i) * kPitch16 + (ec + 16 * j) * 2) =
            make_uint2(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
    }
  __syncthreads();
  if (C_F32)
    store_rows32<TBN, kPitch32, NT, TBM>(smem, Cp, p.ldc, m0, m_end, n0, n_end, p.vec_store, true,
                                         [](int q) { return q; });
  else
    store_rows16<TBM, TBN, kPitch16, NT>(smem, Cp, p.ldc, m0, m_end, n0, n_end, p.vec_store);
}

template <int WM, int WN, int TM, int TN, int U, int NS>
hipError_t launch(NtArgs a, int c_f32, hipStream_t s) {
  constexpr int TBM = 16 * WM * TM, TBN = 16 * WN * TN;
  a.tiles_m = (int)((a.M + TBM - 1) / TBM);
  a.tiles_n = (int)((a.N + TBN - 1) / TBN);
  const dim3 grid((unsigned)((int64_t)a.tiles_m * a.tiles_n)), b(WM * WN * 64);
  if (c_f32 && a.split_stage > 0)
    hipLaunchKernelGGL((gemm_small_kernel<true, true, WM, WN, TM, TN, U, NS>), grid, b, 0, s, a);
  else if (c_f32)
    hipLaunchKernelGGL((gemm_small_kernel<true, false, WM, WN, TM, TN, U, NS>), grid, b, 0, s, a);
  else
    hipLaunchKernelGGL((gemm_small_kernel<false, false, WM, WN, TM, TN, U, NS>), grid, b, 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_small(const NtArgs& a, GemmTile form, int c_f32, hipStream_t s) {
  switch (form) {
    case GemmTile::k128x128: return launch<2, 4, 4, 2, 1, 4>(a, c_f32, s);
    case GemmTile::k128x64: return launch<2, 2, 4, 2, 1, 5>(a, c_f32, s);
    case GemmTile::k64x64: return launch<2, 2, 2, 2, 1, 5>(a, c_f32, s);
    case GemmTile::k32x32: return launch<2, 2, 1, 1, 2, 4>(a, c_f32, s);
    case GemmTile::k16x16: return launch<1, 1, 1, 1, 4, 4>(a, c_f32, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qf
