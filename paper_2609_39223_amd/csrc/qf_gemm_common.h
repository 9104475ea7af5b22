// Shared pieces of the BF16 MFMA GEMM kernels (qf_gemm_nt.hip, qf_gemm_mn.hip): launch arguments,
// tile constants and small device helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qf.h"
#include "qf_codecs.h"
#include "qf_internal.h"

namespace qf {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

constexpr int BK = 64;                          // K depth of a stage
constexpr int kRow = BK * 2;                     // 128 bytes per LDS row
// Dense tile order: groups of kGroupM row tiles, walked column by column (the 9B layer step
// measured 31.2 / 30.2 / 29.5 / 29.9 / 32.0 / 36.4 ms for groups of 1 / 2 / 4 / 8 / 16 / 32).
constexpr int kGroupM = 4;
constexpr int kXcds = 8;
constexpr int64_t kMaxSplitTiles = 128;          // split tiles of the last round, at most

// Fragment-major layout of a B operand [N, K] (K a multiple of 16): block (nb, kb) holds rows
// 32 nb .. 32 nb + 31 and columns 16 kb .. 16 kb + 15 as the 64 lanes' MFMA operands of
// v_mfma_f32_32x32x16_bf16 (lane L: row 32 nb + L % 32, columns 16 kb + 8 (L / 32) .. +7, 16
// bytes), blocks ordered nb-major: element (n, k) at
//   ((n / 32) (K / 16) + k / 16) kBfBlock + ((n % 32) + 32 ((k / 8) % 2)) 8 + k % 8,
// rows past N zero.  A wavefront's operand of one slice and block is one contiguous 1 KB load.
constexpr int kBfBlock = 512;                    // elements per block (64 lanes x 8)
// kDenseAT / kGroupRowsAT: dense / grouped rows, and the launch also writes A^T (NtArgs::at).
enum Mode { kDense = 0, kGroupRows = 1, kGroupK = 2, kDenseAT = 3, kGroupRowsAT = 4 };

struct NtArgs {
  const uint16_t* A;
  const uint16_t* B;
  void* C;
  int64_t lda, ldb, ldc;
  int64_t bstride;        // grouped rows: elements between experts' B
  int64_t M, N, K;
  int tiles_m, tiles_n;
  const int64_t* off;     // grouped rows: [E+1] row offsets
  const int* tile_start;  // grouped rows: [E+1] per-expert tile prefix, then the rows of a tile
  int E;
  // grouped K (per-expert weight gradient): expert e contracts over k in
  // [BK kstart[e], BK kstart[e+1]) and writes C + e cstride; order[] lists experts by
  // decreasing work.  Every XCD owns the same contiguous eighth of each expert's tile grid
  // and runs its share of the experts in that order (see the item mapping in the kernel).
  const int* kstart;
  const int* order;
  int64_t cstride;
  int vec_store;          // C and ldc allow 16-byte stores
  // FP32 split of the last partial round.  Tiles [split_from, tiles) are computed as two
  // K-halves (stages [0, split_stage) and the rest); half h of tile split_from + i writes its
  // 256 x 256 FP32 partial to part[2 i + h].  Work items are laid out per XCD (each XCD runs
  // a contiguous range, see remap_xcd): full_per_xcd whole tiles, then split_per_xcd tiles as
  // 2 halves each, so every XCD ends with a full round of half-length items.
  float* part;
  int split_from, full_per_xcd, split_per_xcd;
  int norot;              // walk K from its start on every XCD (see the kernel's K order)
  int64_t split_stage;
  // kDenseAT / kGroupRowsAT: A^T (row stride ldat) is written as a by-product of the main
  // loop, from the A tiles in LDS (see the kernel).  Dense: A^T [K][M].  Grouped rows: the
  // padded layout of the grouped weight gradient, expert e's rows at columns 64 kstart[e] + i
  // and zeros up to 64 kstart[e+1].
  uint16_t* at;
  int64_t ldat;
  // Packed B (the forward's weight, gemm_nt_kernel's BQ != 0): NVFP4 / MXFP4 codes [N][K/2]
  // (element 2i in the low nibble) and block scales [N][K/16 | K/32], NVFP4's tensor decode
  // scale S at bq_S; or Q4_K blocks [N][K/256][144] at bq_codes.  Each stage's B tile is
  // decoded from these in the main loop (K a multiple of 64).
  const uint8_t* bq_codes;
  const uint8_t* bq_scales;
  const float* bq_S;
};

#define QF_LDS(p) ((__attribute__((address_space(3))) void*)(p))

// 16-byte direct-to-LDS loads: lane l's 16 bytes land at lds + 16 l (lds wave-uniform).
// Reads at voff + soff from a resource whose range ends at the operand's last valid byte (reads
// past it return zeros).  (The global form, global_load_lds, the compiler counts as an LDS access
// of unknown order, which turns the fine-grained lgkmcnt waits of the fragment reads that follow
// into full waits.  Plain functions: device builtins with template-dependent operands keep the
// host pass from emitting the kernel's launch stub.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int64_t bytes) {
  const int64_t n = bytes < 0xFFFFFFFFll ? bytes : 0xFFFFFFFFll;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(uint32_t)n,
                                           0x00020000);
}
__device__ __forceinline__ void dma16_buf(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff,
                                          void* lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, QF_LDS(lds), 16, (int)voff, (int)soff, 0, 0);
}
// Workgroup barrier that orders LDS accesses only: outstanding global stores are not waited
// for (a plain __syncthreads() would drain them).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// 16-byte store of an output row segment.  Output tiles go out non-temporally: they are not
// read again by this launch, and as ordinary stores their lines displace operand panels in L2
// (measured 2-5 % slower on whole launches); split partials, read back right away, stay cached.
__device__ __forceinline__ void store_c16(void* dst, uint4 v, bool nt) {
  if (nt) __builtin_nontemporal_store(u32x4_t{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4_t*>(dst));
  else *reinterpret_cast<uint4*>(dst) = v;
}

// Two FP32 values -> packed bf16 pair (lo in bits 0-15), round to nearest even.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

__device__ __forceinline__ int remap_xcd(int bid, int nb) {
  const int full = nb - nb % kXcds;
  if (bid >= full) return bid;
  return (bid % kXcds) * (full / kXcds) + bid / kXcds;
}

// FP32 split of the last partial round (NtArgs::part): the tile (bid) and K half of work item
// `item`, and the partial it writes.
__device__ __forceinline__ void split_item(const NtArgs& p, int item, int& bid, int& half,
                                           int& pidx) {
  const int per_xcd = p.full_per_xcd + 2 * p.split_per_xcd;
  const int x = item / per_xcd, j = item % per_xcd;
  if (j < p.full_per_xcd) {
    bid = x * p.full_per_xcd + j;
  } else {
    const int i = x * p.split_per_xcd + ((j - p.full_per_xcd) >> 1);
    bid = p.split_from + i;
    half = (j - p.full_per_xcd) & 1;
    pidx = 2 * i + half;
  }
}

// Origin of tile t of an (M, N) output in TBM x TBN tiles: groups of kGroupM tile rows walked
// column by column.
template <int TBM, int TBN>
__device__ __forceinline__ void tile_origin(const NtArgs& p, int t, int64_t& m0, int64_t& n0) {
  const int per_group = kGroupM * p.tiles_n;
  const int first = t / per_group * kGroupM;
  const int gs = min(p.tiles_m - first, kGroupM);
  m0 = (int64_t)(first + (t % per_group) % gs) * TBM;
  n0 = (int64_t)((t % per_group) / gs) * TBN;
}

// A bf16 tile staged in LDS (TBM rows of TBN values, PITCH bytes apart) -> whole-row 16-byte
// stores at C rows em0.., columns en0.. (rows below em_end, columns below en_end).
template <int TBM, int TBN, int PITCH, int NT>
__device__ __forceinline__ void store_rows16(const char* smem, char* Cp, int64_t ldc, int64_t em0,
                                             int64_t em_end, int64_t en0, int64_t en_end,
                                             int vec) {
  constexpr int LPR = TBN / 8, RPP = NT / LPR;   // lanes per row, rows per pass
  const int c8 = (threadIdx.x % LPR) * 8;
  const int64_t gcol = en0 + c8;
#pragma unroll 4
  for (int it = 0; it < (TBM + RPP - 1) / RPP; ++it) {
    const int r = it * RPP + (int)threadIdx.x / LPR;
    if (TBM % RPP != 0 && r >= TBM) break;       // more lanes than the tile has segments
    const int64_t grow = em0 + r;
    if (grow >= em_end || gcol >= en_end) continue;
    const uint4 v = *reinterpret_cast<const uint4*>(smem + r * PITCH + c8 * 2);
    uint16_t* dst = reinterpret_cast<uint16_t*>(Cp) + grow * ldc + gcol;
    if (vec && gcol + 8 <= en_end) {
      store_c16(dst, v, true);
    } else {
      const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
      for (int e = 0; e < 8 && gcol + e < en_end; ++e)
        dst[e] = (uint16_t)(wv[e >> 1] >> (16 * (e & 1)));
    }
  }
}

// The same for 128 FP32 rows staged in LDS; row(q) is the tile row of LDS row q.
template <int TBN, int PITCH, int NT, int ROWS = 128, class Row>
__device__ __forceinline__ void store_rows32(const char* smem, char* Cp, int64_t ldc, int64_t em0,
                                             int64_t em_end, int64_t en0, int64_t en_end, int vec,
                                             bool nt, Row row) {
  constexpr int LPR = TBN / 4, RPP = NT / LPR;
  const int c4 = (threadIdx.x % LPR) * 4;
  const int64_t gcol = en0 + c4;
#pragma unroll 4
  for (int it = 0; it < (ROWS + RPP - 1) / RPP; ++it) {
    const int q = it * RPP + (int)threadIdx.x / LPR;
    if (ROWS % RPP != 0 && q >= ROWS) break;
    const int64_t grow = em0 + row(q);
    if (grow >= em_end || gcol >= en_end) continue;
    const uint4 v = *reinterpret_cast<const uint4*>(smem + q * PITCH + c4 * 4);
    float* dst = reinterpret_cast<float*>(Cp) + grow * ldc + gcol;
    if (vec && gcol + 4 <= en_end) {
      store_c16(dst, v, nt);
    } else {
      const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
      for (int e = 0; e < 4 && gcol + e < en_end; ++e) dst[e] = __uint_as_float(wv[e]);
    }
  }
}

// qf_gemm_mn.hip: `items` work items of 256 x 256 tiles with at least one K-as-rows operand.
hipError_t launch_gemm_mn_tiles(const NtArgs& a, int items, int a_mn, int b_mn, int c_f32,
                                hipStream_t s);

// Tiles of the dense k-contiguous product: the main kernel's two (qf_gemm_nt.hip) and the small
// kernel's (qf_gemm_small.hip).  All but k256x256 walk K from its start (NtArgs::norot).
enum class GemmTile { k256x256, k256x128, k128x128, k128x64, k64x64, k32x32, k16x16 };
hipError_t launch_gemm_small(const NtArgs& a, GemmTile form, int c_f32, hipStream_t s);

}  // namespace qf
