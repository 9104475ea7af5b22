// NT BF16 MFMA GEMM for gfx950: C[m, n] = sum_k A[m, k] * B[n, k], both operands k-contiguous.
//
// Every product of the quantization-aware layer is issued in this form (the backward's
// transposed operands come from the transpose kernel), so this is the one kernel that carries
// the layer's FLOPs:
//   forward  Y  = A_hat W_hat^T        A = A_hat [M, K],   B = W_hat [N, K]
//   dX          = dY W_hat             A = dY [M, N],      B = W_hat^T [K, N]
//   dW          = dY^T A_hat           A = dY^T [N, M],    B = A_hat^T [K, M]
//
// Design (256 x 256 block tile, 256 x 128 where that fills the chip better, 128 x 256 for experts
// with few rows):
//  - 4 wavefronts, one per SIMD, each owning a 128 x 128 (128 x 64) sub-tile as 16 x 16
//    v_mfma_f32_16x16x32_bf16 accumulators (256 / 128 AGPRs).  What bounds the full launches is
//    power: at 8192 x 14336 x 4096 the chip holds 1.84 GHz in this loop with the MFMA pipes 80 %
//    busy, against 1.65 GHz and 82 % with the same loop built on 32 x 32 x 16 MFMAs (counter
//    runs), and takes 617 us (1.56 PFLOP/s) against 664, to the same bits.
//  - K advances in 64-deep stages, double-buffered in LDS (2 x 64 KB).  A stage row is 128
//    bytes, so every global request is a whole 128-byte cache line (32-deep stages fetch half
//    lines and double the L2 request count).
//  - Operands move global -> LDS with direct-to-LDS loads (no staging registers, no ds_write),
//    16 loads of 8 rows each per wavefront and stage.  The loads of stage s+1 are spread over
//    two slices (the second of step s-1, right after the barrier that frees its buffer, and the
//    first of step s), so the memory pipe sees a steady stream rather than a burst.
//  - MFMAs are interleaved with the fragment reads of the next 32-deep slice and the
//    direct-to-LDS loads, at most one of each per MFMA, so the LDS and memory pipes work while
//    the MFMA pipe is busy (copies every second or third MFMA instead of every fourth: 2 to 6 %
//    slower launches).  One barrier per step, between its two slices: it publishes stage
//    s+1 (all loads waited) and retires every read of stage s (so stage s+2 may overwrite it).
//  - LDS rows hold 64 bf16 (8 chunks of 16 bytes); chunk c of row r sits at slot
//    c ^ ((r >> 1) & 7), so the 16 rows a fragment read serves in one pass fall on 16
//    distinct 16-byte bank groups.
//  - Rows past the matrix edge load the last valid row (their outputs are never stored); a
//    partial last k stage goes through a masked register path.
//  - The epilogue stages the tile through LDS (rows padded so both half-waves of a write hit
//    different banks) and writes whole rows with 16-byte stores; FP32 tiles go in two halves.
//  - Block ids are remapped so each XCD (own L2) works on a contiguous group of tiles, and
//    each XCD walks K from its own rotated start (HBM channel spread).
//  - Optionally (kDenseAT / kGroupRowsAT, the backward's dX = dY W_hat, dense or per expert)
//    the launch also writes A^T: each staged k stage of A is split into 16 pieces of 4 k-rows,
//    each owned by one tile of the row panel, which gathers its piece from LDS before the
//    step's barrier and stores it as whole 128-byte rows after it.  That replaces a separate
//    transpose pass over dY (grouped: into the padded per-expert columns of the weight
//    gradient, zeros included).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "qf_gemm_common.h"

namespace qf {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int BM = 256, BN = 256;                // the main tile

// c += y x^T (16 x 16 x 32).  Inline assembly, because it ties the accumulator to one register:
// with the builtin the allocator, all 256 accumulation registers in use, moved accumulators
// through vector registers in the loop (56 moves per 256 MFMAs in the plain form, 580 with
// spills where the loop also writes A^T); tied, none.  The compiler knows the operands (it waits
// for the fragment reads) but not that this is an MFMA, so the wait states the hardware wants
// from software are acc_settle's: two between a vector write of an operand and the MFMA that
// reads it (fragments come from LDS or memory only, accumulators are initialized before the
// loop), and those of an eight-pass MFMA between its write and any other read of it.
__device__ __forceinline__ void mfma16(f32x4_t& c, const bf16x8_t& x, const bf16x8_t& y) {
  asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
}

// The wait states between an MFMA and any other access to its result, for the copies the
// compiler may place where the main loop and its last steps meet.
__device__ __forceinline__ void mfma_wait() { asm volatile("s_nop 15\n\ts_nop 15"); }

// Pins the accumulators at this point, with wait states after their initialization (BEGIN) or
// before their first use outside the MFMAs (volatile statements keep their order).
template <bool BEGIN, int TM, int TN>
__device__ __forceinline__ void acc_settle(f32x4_t (&acc)[TM][TN]) {
  if (!BEGIN) mfma_wait();
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
  if (BEGIN) asm volatile("s_nop 7");
}

// A value that all lanes share, in scalar registers (loaded through a pointer, the compiler may keep
// it in vector registers, and then wraps every buffer operation whose resource depends on it in a
// loop over the lanes' values).
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
  return ((int64_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | lo;
}

// 16-byte LDS store that does not wait for direct-to-LDS copies under way: before an ordinary one the
// compiler waits for them all, as they might write the same bytes (four times a step where B is
// decoded: 32768 x 24576 x 4096 NVFP4, quantizer and GEMM, 8936 us, 6115 with this store).  Only for
// bytes that no copy in flight writes.  The compiler does not count it in lgkmcnt: the next barrier's
// wait has to be lgkmcnt(0).
__device__ __forceinline__ void lds_store16(char* dst, u32x4_t v) {
  asm volatile("ds_write_b128 %0, %1" : : "v"((uint32_t)(uintptr_t)QF_LDS(dst)), "v"(v) : "memory");
}

// f(0), f(1), .. f(N - 1) with compile-time indices (std::integral_constant arguments)
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// LDS bytes of a tile: two stages (and the prefetches' landing place), or its bf16 form padded
constexpr int nt_smem_bytes(int TM, int TN, bool PF) {
  const int stages = 2 * 32 * (TM + TN) * kRow + (PF ? 1024 : 0), c16 = 32 * TM * (64 * TN + 16);
  return stages > c16 ? stages : c16;
}

// TM x TN: 16 x 16 accumulator blocks of a wavefront's sub-tile; the 2 x 2 wavefronts of a
// workgroup own a 32 TM x 32 TN tile (8 x 8: 256 x 256; 8 x 4: 256 x 128; 4 x 8: 128 x 256).
//
// BQ != 0 (QF_FMT_NVFP4 / MXFP4 / Q4K; 256-column tile, dense or per expert, bf16 C): B is the
// packed quantized weight (the experts' back to back) instead of a bf16 matrix.  Each lane owns one B row of its
// wavefront's 64 (row 64 w + lane) and, one step ahead, loads that row's codes and scales for
// a stage into registers (32 bytes of codes plus 4 / 2 scale bytes, or the Q4_K block's 16-byte
// header and 32 code bytes); in the next step it decodes them with the quantizers' own decode
// functions (so the B tile holds x_hat bit for bit) and writes the 8 chunks into the stage's
// LDS buffer with 16-byte writes, interleaved with that step's MFMAs, before the barrier that
// publishes the stage.  A keeps its direct-to-LDS loads.
//
// BF (256 x 256 tile, dense modes, K a multiple of 64): B comes in the
// fragment-major layout (see kBfBlock) straight from memory into the MFMA operand registers,
// one load of four 256-byte runs per 16-row block and 32-deep slice, and never enters LDS: LDS
// then carries only A (its direct-to-LDS copies and fragment reads), half of the traffic of
// the form above, which is the budget the MFMAs wait on.  Each B fragment of stage s+1 is
// loaded right after the last MFMA that uses the same register for stage s, so it has a whole
// step to arrive; A's copies of stage s+1 all go out at the start of step s, ahead of every B
// load of the step, and the barrier waits for them while leaving that step's B loads in flight.
//
// AT2 (A^T modes): a tile may own two A^T pieces per stage (fewer than 16 tile columns); without
// it the launch has at least 16 and a tile owns at most one.
template <bool C_F32, int MODE, int TM, int TN, int BQ, bool BF, bool AT2, bool PF>
__device__ __forceinline__ void gemm_nt_tile(const NtArgs& p, char* smem) {
  static_assert((TM == 8 && (TN == 8 || TN == 4)) || (TM == 4 && TN == 8 && MODE == kGroupRows),
                "256-row tiles of 256 or 128 columns; per expert also 128 rows by 256 columns");
  static_assert(BQ == 0 || (TN == 8 && (MODE == kDense || MODE == kGroupRows) && !C_F32),
                "packed B: 256-column bf16 forms without A^T");
  static_assert(!BF || (TN == 8 && BQ == 0 && (MODE == kDense || MODE == kDenseAT)),
                "fragment-major B: the dense 256 x 256 forms");
  constexpr int BM = 32 * TM, BN = 32 * TN;
  constexpr int kOpStage = BM * kRow;            // A's LDS bytes of a stage; B's follow
  constexpr int kStage = (BM + BN) * kRow;
  constexpr int kPitch16 = BN * 2 + 16;          // epilogue LDS row pitch, bf16 tile
  constexpr int kPitch32 = BN * 4 + 16;          // epilogue LDS row pitch, FP32 half tile
  constexpr int kSmem = nt_smem_bytes(TM, TN, PF);
  static_assert(BM / 2 * kPitch32 <= kSmem, "the FP32 half tile fits the stages' LDS");
  // direct-to-LDS loads per wavefront per stage: TM of A, then TN of B (packed or
  // fragment-major B: A's only)
  constexpr int NLD = (BQ != 0 || BF) ? TM : TM + TN;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform (scalar) index
  const int wm = w >> 1, wn = w & 1;
  constexpr bool DENSE = MODE == kDense || MODE == kDenseAT;
  constexpr bool AT = MODE == kDenseAT || MODE == kGroupRowsAT;
  static_assert(!AT || !C_F32, "A^T output: bf16 form");
  // stage s+1's loads: L0 in the second slice of step s-1, the rest in the first of step s
  // (fragment-major B: all of A's in the latter)
  constexpr int L0 = BF ? NLD : AT || BQ != 0 ? NLD / 2 : NLD / 4 * 3;
  constexpr int CSTEP = TM == 4 ? 2 : TN / 2;    // MFMAs per copy issued
  static_assert((L0 > NLD - L0 ? L0 : NLD - L0) * CSTEP <= TM * TN, "a slice holds its copies");
  // stages between a prefetch and the stage being multiplied: us with 2 / 3 / 4, FP32 6144 x 4096
  // x 32768 1281 / 1192 / 1171, writing A^T 32768 x 4096 x 24576 4518 / 4561 / 4580, the expert
  // layer's down projection (forward + backward) 8521 / 8542 / 8646
  constexpr int kPfDist = DENSE && C_F32 ? 4 : 2;
  static_assert(!PF || (BQ == 0 && !BF), "prefetch: both operands through LDS");
  const int item = remap_xcd(blockIdx.x, gridDim.x);
  int bid = item, half = -1, pidx = 0;
  if (DENSE && C_F32 && p.part != nullptr) split_item(p, item, bid, half, pidx);

  const uint16_t* Bp = p.B;
  int64_t m0, m_end, n0;
  int ks0 = 0, ks1 = (int)(p.K / BK);            // stage range of this item
  int64_t cofs = 0;                              // element offset of this item's C
  int64_t bq_e = 0;                              // expert of this item (packed B)
  // A^T columns of this tile's first row and the end of its A^T range: rows whose column is
  // below at_end but lie past the operand get zeros (grouped padding)
  int64_t at_col0 = 0, at_end = 0;
  if (DENSE || MODE == kGroupK) {
    int t = bid;
    if (MODE == kGroupK) {
      // Block b runs on XCD x = b % 8 as that XCD's item j = b / 8.  XCD x owns tiles
      // [x tpe / 8, (x + 1) tpe / 8) of every expert; its items walk the experts in order[]
      // (decreasing work), cmax = ceil(tpe / 8) items per expert, the surplus ones empty.  So
      // the 8 XCDs carry equal work however skewed the routing is, and each XCD's CUs take
      // the largest tiles first.
      const int tpe = p.tiles_m * p.tiles_n;
      const int cmax = (tpe + kXcds - 1) / kXcds;
      const int x = blockIdx.x % kXcds, j = blockIdx.x / kXcds;
      const int lo = x * tpe / kXcds, hi = (x + 1) * tpe / kXcds;
      t = lo + j % cmax;
      if (t >= hi) return;                         // uniform over the block
      const int e = p.order[j / cmax];
      ks0 = p.kstart[e];
      ks1 = p.kstart[e + 1];
      cofs = (int64_t)e * p.cstride;
    }
    tile_origin<BM, BN>(p, t, m0, n0);
    m_end = p.M;
    at_col0 = m0;
    at_end = (m_end + 7) / 8 * 8;                // (rows past the last of a ragged M: zeros)
  } else {
    // The grid is sized for the most row tiles any routing can need; the real count is
    // tile_start[E].  Block b runs on XCD x = b % 8 as its item j = b / 8, and XCD x takes the
    // contiguous range [x per, (x + 1) per) of the real items (per = ceil(items / 8)), so the
    // XCDs get equal shares and their 32 CUs share the expert weight panels in their L2.
    const int items = __builtin_amdgcn_readfirstlane(p.tile_start[p.E]) * p.tiles_n;
    const int per = (items + kXcds - 1) / kXcds;
    const int j = blockIdx.x / kXcds, it = (blockIdx.x % kXcds) * per + j;
    if (j >= per || it >= items) return;         // uniform over the block
    const int mt = it / p.tiles_n, tn = it % p.tiles_n;
    int lo = 0, hi = p.E;                        // tile_start[e] <= mt < tile_start[e+1]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (p.tile_start[mid] <= mt) lo = mid; else hi = mid;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    m0 = uniform64(p.off[lo] + (int64_t)(mt - p.tile_start[lo]) * BM);
    m_end = uniform64(p.off[lo + 1]);
    n0 = (int64_t)tn * BN;
    if (AT) {
      at_col0 = 64 * (int64_t)p.kstart[lo] + (m0 - p.off[lo]);
      at_end = 64 * (int64_t)p.kstart[lo + 1];
    }
    Bp += (int64_t)lo * p.bstride;
    bq_e = lo;
  }
  const int64_t n_end = p.N, K = p.K;

  // ---- this lane's loads ----------------------------------------------------------------------
  // Wavefront w loads rows 8 TM w .. of A (loads 0 .. TM - 1, 8 rows = 1 KB each) and rows 8 TN w
  // .. of B (loads TM ..).  A stage is BM + BN rows of 128 bytes: load q covers 8 rows from R,
  // lane l lands at row R + l / 8, slot l % 8 and so fetches logical chunk
  // (l % 8) ^ ((row >> 1) % 8) = (l % 8) ^ ((4 (q % 2) + l / 16) % 8).
  const char* gb[2];
  __amdgpu_buffer_rsrc_t rs[2];
  uint32_t goff[NLD];
#pragma unroll
  for (int op = 0; op < 2; ++op) {
    if ((BQ != 0 || BF) && op == 1) continue;    // packed / fragment-major B: registers
    const int64_t ld = op ? p.ldb : p.lda;
    const int64_t r0 = op ? n0 : m0;
    const int64_t rlim = (op ? n_end : m_end) - r0 - 1;   // last valid row
    gb[op] = reinterpret_cast<const char*>((op ? Bp : p.A) + r0 * ld);
    rs[op] = make_rsrc(gb[op], (rlim * ld + K) * 2);
    const int nq = op ? TN : TM, q0 = op ? TM : 0;
#pragma unroll
    for (int q = 0; q < nq; ++q) {
      const int64_t row = (w * nq + q) * 8 + (lane >> 3);
      const int64_t rc = row < rlim ? row : rlim;
      const int c = (lane & 7) ^ ((4 * (q & 1) + (lane >> 4)) & 7);
      goff[q0 + q] = (uint32_t)((rc * ld + c * 8) * 2);
    }
  }
  // ---- L2 prefetch (PF) -------------------------------------------------------------------
  // pf_off: this lane's 16 bytes of one eighth of A's rows and two of one quarter of B's rows of
  // a stage (the tiles of an XCD that run together share them, see the main loop).
  uint32_t pf_off[3];
  if (PF) {
    const int64_t ra = m_end - m0 - 1, rb = n_end - n0 - 1;
    const int64_t a = ((n0 / BN) & 7) * (BM / 8) + w * (BM / 32) + (lane >> 3);
    pf_off[0] = (uint32_t)(((a < ra ? a : ra) * p.lda + (lane & 7) * 8) * 2);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t b = ((m0 / BM) & 3) * (BN / 4) + w * (BN / 16) + h * 8 + (lane >> 3);
      pf_off[1 + h] = (uint32_t)(((b < rb ? b : rb) * p.ldb + (lane & 7) * 8) * 2);
    }
  }
  auto lds_of = [&](int q) {
    return q < TM ? (w * TM + q) * 1024 : kOpStage + (w * TN + q - TM) * 1024;
  };

  // ---- packed B (BQ != 0): this lane's row and its per-stage loads -------------------------
  // Row brow = 64 w + lane of the tile (rows past N decode the last valid row; their outputs
  // are never stored).  Registers of one stage: c0, c1 = the 32 code bytes (element 2i in the
  // low nibble; Q4_K: byte l holds sub-block 2g's element l low and 2g+1's high), sc = the
  // block scales (NVFP4 4 bytes, MXFP4 2) or hd = the Q4_K block header (d, dmin, 12 scale bytes).
  struct BqRegs {
    uint4 c0, c1, hd;
    uint32_t sc;
  };
  const int brow = w * 64 + lane;
  const uint8_t* bq_row = nullptr;
  const uint8_t* bq_srow = nullptr;
  float bq_S = 0.0f;
  if (BQ != 0) {
    const int64_t gr = bq_e * n_end + (n0 + brow < n_end ? n0 + brow : n_end - 1);
    if (BQ == QF_FMT_Q4K) {
      bq_row = p.bq_codes + gr * (K / 256) * 144;
    } else {
      bq_row = p.bq_codes + gr * (K / 2);
      bq_srow = p.bq_scales + gr * (K / (BQ == QF_FMT_NVFP4 ? 16 : 32));
    }
    if (BQ == QF_FMT_NVFP4) bq_S = p.bq_S[bq_e];    // the quantizer's S = fl(g / 2688)
  }
  auto bq_load = [&](int64_t se, BqRegs& r) __attribute__((always_inline)) {
    if (BQ == QF_FMT_Q4K) {
      const uint8_t* blk = bq_row + (se >> 2) * 144;
      r.hd = *reinterpret_cast<const uint4*>(blk);
      r.c0 = *reinterpret_cast<const uint4*>(blk + 16 + 32 * (se & 3));
      r.c1 = *reinterpret_cast<const uint4*>(blk + 32 + 32 * (se & 3));
    } else {
      r.c0 = *reinterpret_cast<const uint4*>(bq_row + se * 32);
      r.c1 = *reinterpret_cast<const uint4*>(bq_row + se * 32 + 16);
      if (BQ == QF_FMT_NVFP4) r.sc = *reinterpret_cast<const uint32_t*>(bq_srow + se * 4);
      else r.sc = *reinterpret_cast<const uint16_t*>(bq_srow + se * 2);
    }
  };
  // x_hat of logical chunk c (elements 8c .. 8c+7 of the stage) into LDS buffer buf.
  auto bq_decode = [&](const BqRegs& r, int64_t se, int c, int buf) __attribute__((always_inline)) {
    const uint32_t cw[8] = {r.c0.x, r.c0.y, r.c0.z, r.c0.w, r.c1.x, r.c1.y, r.c1.z, r.c1.w};
    uint32_t o[4];
    if (BQ == QF_FMT_NVFP4) {
      // (with a non-finite tensor scale the decoded NaN operands may differ from the
      // quantizer's x_hat in NaN sign and payload only, which the NaN sums do not show)
      codec::nvfp4_decode8_finite(
          cw[c], codec::nvfp4_block_scale(bq_S, (r.sc >> (8 * (c >> 1))) & 0xFFu), o);
    } else if (BQ == QF_FMT_MXFP4) {
      codec::mxfp4_decode8(cw[c], (r.sc >> (8 * (c >> 2))) & 0xFFu, o);
    } else {
      // sub-block j = 2 (se % 4) + (c >= 4): its 6-bit scale and min from the header
      const int j = 2 * (int)(se & 3) + (c >> 2);
      const int jj = j & 3, sh = 8 * jj;
      uint32_t ls, lm;
      if (j < 4) {
        ls = (r.hd.y >> sh) & 63u;
        lm = (r.hd.z >> sh) & 63u;
      } else {
        ls = ((r.hd.w >> sh) & 15u) | (((r.hd.y >> (sh + 6)) & 3u) << 4);
        lm = ((r.hd.w >> (sh + 4)) & 15u) | (((r.hd.z >> (sh + 6)) & 3u) << 4);
      }
      const float t1 = codec::f16_value(r.hd.x & 0xFFFFu) * (float)ls;
      const float t2 = codec::f16_value(r.hd.x >> 16) * (float)lm;
      const int b = (c & 3) * 2;                  // code bytes 8 (c % 4) .. +7
      const uint32_t sh4 = c >= 4 ? 4u : 0u;      // sub-block 2g + 1 in the high nibbles
      const uint32_t qw[2] = {(cw[b] >> sh4) & 0x0F0F0F0Fu, (cw[b + 1] >> sh4) & 0x0F0F0F0Fu};
      codec::q4k_decode8(qw, t1, t2, o);
    }
    *reinterpret_cast<uint4*>(smem + buf * kStage + kOpStage + brow * kRow +
                              ((c ^ ((brow >> 1) & 7)) << 4)) = make_uint4(o[0], o[1], o[2], o[3]);
  };
  BqRegs bq_cur{}, bq_nxt{};
  // The main loop decodes a stage as a chain of small operations, each after an MFMA of its own
  // (the first half of the chunks in the second slice of the step before, the rest in the first
  // slice), so that no gap between two MFMAs holds more than a few VALU instructions (one
  // wavefront per SIMD: nothing else issues while this one decodes).
  //   NVFP4, 48 operations: per chunk c, the block decode scale D (even c), the four element
  //          pairs (E2M1 -> FP32, x D, bf16 pack), the 16-byte LDS write.
  //   MXFP4, 24: per chunk, pairs 0-1 with the E8M0 scale, pairs 2-3, the
  //          NaN-block select and the write.
  //   Q4_K, 43: the super-block's d and dmin, the two sub-blocks' step t1 and offset t2, then
  //          per chunk four element pairs (the first also extracts the chunk's nibbles) and
  //          the write.
  // The arithmetic is the decode functions' (codec::*_decode8), split up.
  float bq_D = 0.0f, bq_d = 0.0f, bq_dmin = 0.0f, bq_t1[2] = {0.0f, 0.0f}, bq_t2[2] = {0.0f, 0.0f};
  uint32_t bq_o[4] = {0, 0, 0, 0}, bq_qw[2] = {0, 0}, bq_x = 0;
  auto bq_word = [&](const BqRegs& r, int c) __attribute__((always_inline)) -> uint32_t {
    switch (c) {
      case 0: return r.c0.x; case 1: return r.c0.y; case 2: return r.c0.z; case 3: return r.c0.w;
      case 4: return r.c1.x; case 5: return r.c1.y; case 6: return r.c1.z; default: return r.c1.w;
    }
  };
  auto bq_store = [&](int c, int buf) __attribute__((always_inline)) {
    lds_store16(smem + buf * kStage + kOpStage + brow * kRow + ((c ^ ((brow >> 1) & 7)) << 4),
                u32x4_t{bq_o[0], bq_o[1], bq_o[2], bq_o[3]});
  };
  constexpr int kBqOps = BQ == QF_FMT_NVFP4 ? 48 : BQ == QF_FMT_MXFP4 ? 24 : 43;
  auto bq_op = [&](const BqRegs& r, int64_t se, int u, int buf) __attribute__((always_inline)) {
    if (BQ == QF_FMT_NVFP4) {
      const int c = u / 6, k = u % 6;
      const uint32_t cw = bq_word(r, c);
      if (k == 0) {
        if ((c & 1) == 0) bq_D = codec::nvfp4_block_scale(bq_S, (r.sc >> (8 * (c >> 1))) & 0xFFu);
      } else if (k <= 4) {
        // (with a non-finite tensor scale the decoded NaN operands may differ from the
        // quantizer's x_hat in NaN sign and payload only, which the NaN sums do not show)
        codec::f32x2_t v;
        switch (k) {
          case 1: v = codec::e2m1_pair<0>(cw); break;
          case 2: v = codec::e2m1_pair<1>(cw); break;
          case 3: v = codec::e2m1_pair<2>(cw); break;
          default: v = codec::e2m1_pair<3>(cw); break;
        }
        bq_o[k - 1] = codec::bf16x2_rne_nonnan(v.x * bq_D, v.y * bq_D);
      } else {
        bq_store(c, buf);
      }
    } else if (BQ == QF_FMT_MXFP4) {
      const int c = u / 3, k = u % 3;
      const uint32_t cw = bq_word(r, c);
      if (k == 0) bq_x = (r.sc >> (8 * (c >> 2))) & 0xFFu;
      const float sc = codec::e8m0_scale(bq_x);
      if (k == 0) {
        bq_o[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(cw, sc, 0));
        bq_o[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(cw, sc, 1));
      } else if (k == 1) {
        bq_o[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(cw, sc, 2));
        bq_o[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(cw, sc, 3));
      } else {
        const bool nan = bq_x == 0xFFu;                // (codec::mxfp4_decode8's NaN block)
#pragma unroll
        for (int q = 0; q < 4; ++q) bq_o[q] = nan ? 0x7FC07FC0u : bq_o[q];
        bq_store(c, buf);
      }
    } else {
      if (u == 0) {
        bq_d = codec::f16_value(r.hd.x & 0xFFFFu);        // d and dmin of the super-block
        bq_dmin = codec::f16_value(r.hd.x >> 16);
      } else if (u < 3) {
        // sub-block j = 2 (se % 4) + u - 1: its 6-bit scale and min from the header
        const int j = 2 * (int)(se & 3) + u - 1;
        const int sh = 8 * (j & 3);
        uint32_t ls, lm;
        if (j < 4) {
          ls = (r.hd.y >> sh) & 63u;
          lm = (r.hd.z >> sh) & 63u;
        } else {
          ls = ((r.hd.w >> sh) & 15u) | (((r.hd.y >> (sh + 6)) & 3u) << 4);
          lm = ((r.hd.w >> (sh + 4)) & 15u) | (((r.hd.z >> (sh + 6)) & 3u) << 4);
        }
        bq_t1[u - 1] = bq_d * (float)ls;
        bq_t2[u - 1] = bq_dmin * (float)lm;
      } else {
        const int c = (u - 3) / 5, k = (u - 3) % 5, h = c >> 2;
        if (k == 0) {
          const int b = (c & 3) * 2;                // code bytes 8 (c % 4) .. +7
          const uint32_t sh4 = h ? 4u : 0u;         // sub-block 2g + 1 in the high nibbles
          bq_qw[0] = (bq_word(r, b) >> sh4) & 0x0F0F0F0Fu;
          bq_qw[1] = (bq_word(r, b + 1) >> sh4) & 0x0F0F0F0Fu;
        }
        if (k < 4) {
          // elements 2k, 2k + 1: bf16(fl(t1 q - t2)) as in codec::q4k_decode8
          const uint32_t q = bq_qw[k >> 1] >> (16 * (k & 1));
          const float a0 = __builtin_fmaf(bq_t1[h], (float)(q & 0xFFu), -bq_t2[h]);
          const float a1 = __builtin_fmaf(bq_t1[h], (float)((q >> 8) & 0xFFu), -bq_t2[h]);
          bq_o[k] = codec::bf16x2_rne_nonnan(a0, a1);
        } else {
          bq_store(c, buf);
        }
      }
    }
  };

  // ---- fragment offsets ----------------------------------------------------------------------
  // 32-deep slice kk, fragment i (16 rows of 128 bytes): lane l holds row l % 16, columns
  // 8 (l / 16) .. +7 of the slice, at fo[kk] + i * 2048; fragment rows start 16-aligned, so the
  // swizzle term (row >> 1) & 7 is (lane >> 1) & 7.
  int foa[2], fob[2];
  {
    const int ra = wm * (16 * TM) + (lane & 15), rb = wn * (16 * TN) + (lane & 15);
    const int sw = (lane >> 1) & 7;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int c = 4 * x + (lane >> 4);
      foa[x] = ra * kRow + ((c ^ sw) << 4);
      fob[x] = kOpStage + rb * kRow + ((c ^ sw) << 4);
    }
  }

  f32x4_t acc[TM][TN];
  bf16x8_t fa[2][TM], fb[2][TN];
  // Fragment-major B (BF): fbr[kk][j] holds the B fragment of 32-deep slice kk and 16-row
  // block j of this wavefront's 128 columns for the stage in use.  Blocks 2 jj and 2 jj + 1 are
  // the halves of the layout's 32-row block jj, whose fragments start at bf_base[jj]; slice kk
  // of global stage se is kBfBlock elements further per 16 columns, i.e. per (4 se + 2 kk).
  bf16x8_t fbr[BF ? 2 : 1][BF ? TN : 1];
  const uint16_t* bf_base[BF ? TN / 2 : 1];
  if (BF) {
    const int64_t nblocks = (p.N + 31) / 32, kblocks = p.K / 16;
#pragma unroll
    for (int jj = 0; jj < TN / 2; ++jj) {
      int64_t nb = (n0 + wn * 128) / 32 + jj;
      nb = nb < nblocks ? nb : nblocks - 1;      // blocks past N: outputs never stored
      bf_base[jj] = p.B + (nb * kblocks + (lane >> 5)) * kBfBlock +
                    ((lane & 15) + 32 * ((lane >> 4) & 1)) * 8;
    }
  }
  auto bf_load = [&](int64_t se, int kk, int j) __attribute__((always_inline)) {
    if (BF)
      fbr[kk][j] = *reinterpret_cast<const bf16x8_t*>(bf_base[j >> 1] + (se * 4 + 2 * kk) * kBfBlock +
                                                      (j & 1) * 128);
  };

  // K order: the stages of this item's range [ks0, ks1) are visited rotated by an offset that
  // depends on the XCD (blockIdx.x % 8).  The 32 CUs of an XCD stay in step, so the panels
  // they share still meet in its L2, but the eight XCDs stream from eight different k offsets:
  // with row strides that are large powers of two, k-aligned requests from all CUs otherwise
  // pile onto the same HBM channels.  Each tile's sum order is fixed, so results are
  // deterministic.
  // (Stage indices are 32-bit: fewer scalar instructions in the main loop's issue slots.)
  if (half == 1) ks0 = (int)p.split_stage;
  if (half == 0) ks1 = (int)p.split_stage;
  const int klen = ks1 > ks0 ? ks1 - ks0 : 1;
  const int krot = p.norot ? 0 : (int)(blockIdx.x % kXcds) * (klen / kXcds);
  // global stage of loop stage s
  auto gstage = [&](int s) __attribute__((always_inline)) -> int {
    const int se = s + krot;
    return se >= ks1 ? se - klen : se;
  };
  // load q of global stage se into buffer buf
  auto dma = [&](int se, int buf, int q) __attribute__((always_inline)) {
    dma16_buf(rs[q < TM ? 0 : 1], goff[q], (uint32_t)se * (uint32_t)kRow,
              smem + buf * kStage + lds_of(q));
  };
  // Fragment read r of a slice, in the order the slice's MFMAs consume them: A0, B0 .., A1 ...
  auto read_one = [&](const char* st, int kk, int r, bf16x8_t* a, bf16x8_t* b) __attribute__((always_inline)) {
    if (r == 0 || r > TN) {
      const int i = r == 0 ? 0 : r - TN;
      a[i] = *reinterpret_cast<const bf16x8_t*>(st + foa[kk] + i * 2048);
    } else if (!BF) {
      b[r - 1] = *reinterpret_cast<const bf16x8_t*>(st + fob[kk] + (r - 1) * 2048);
    }
  };
  auto read_all = [&](const char* st, int kk, bf16x8_t* a, bf16x8_t* b) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < TM + TN; ++r) read_one(st, kk, r, a, b);
  };
  // ---- A^T output (kDenseAT, kGroupRowsAT) ---------------------------------------------------
  // A stage's A^T is 16 pieces: piece u is k columns 4 u .. 4 u + 3 over the tile's 256 rows, so
  // each of its rows of A^T is written as whole 128-byte lines, each line by one store.  Piece
  // u of global stage se belongs to tile column (16 se + u) mod tiles_n, so with tiles_n >= 8 a
  // tile has at most two pieces per stage.  at_read gathers this lane's part of piece u from
  // the stage in LDS (rows r0 .. r0 + 3, r0 = 64 w + 4 (l % 16), of k column kc = 4 u + l / 16;
  // four 2-byte reads through the row swizzle) before the step's barrier; at_store writes
  // those 8 bytes to A^T row se * 64 + kc, columns at_col0 + r0 .. +3 (at_col0 = m0 dense, the
  // padded column of the tile's first row grouped), after it, so the store has a whole step to
  // complete before the next barrier's wait.  Rows past the operand store zeros while their
  // column is below at_end (an expert's padding) and nothing beyond it.  Stores go through a
  // buffer resource over the stage's rows of A^T: lanes with nothing to store (or columns at
  // or past kvalid) get an offset beyond its range, which the hardware drops.  (Plain LDS reads:
  // the transposing read builtin makes the compiler wait for every direct-to-LDS load in
  // flight first.)
  const int64_t at_tn = n0 / BN;                 // this tile's column
  const int at_r = w * 64 + 4 * (lane & 15), at_c = lane >> 4;
  // (the four values stay unpacked until the store: packing them at the read would make the
  // wavefront wait for the reads there)
  auto at_read = [&](const char* st, int u) __attribute__((always_inline)) -> u32x4_t {
    const int kc = 4 * u + at_c;
    u32x4_t h;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = at_r + e;
      h[e] = *reinterpret_cast<const uint16_t*>(
          st + row * kRow + ((((kc >> 3) ^ (row >> 1)) & 7) << 4) + (kc & 7) * 2);
    }
    return h;
  };
  // byte offset of this lane's 8 bytes of piece 0 within a stage's rows of A^T (below 2^31)
  const int at_off = (int)(((int64_t)at_c * p.ldat + at_col0 + at_r) * 2);
  const int at_ld8 = (int)(p.ldat * 8);          // bytes of 4 rows of A^T
  // data rows of the four, as masks of the packed values
  const uint32_t at_m01 = (m0 + at_r < m_end ? 0xFFFFu : 0u) | (m0 + at_r + 1 < m_end ? 0xFFFF0000u : 0u);
  const uint32_t at_m23 = (m0 + at_r + 2 < m_end ? 0xFFFFu : 0u) | (m0 + at_r + 3 < m_end ? 0xFFFF0000u : 0u);
  const bool at_zok = at_col0 + at_r < at_end;     // data or zero-padding columns
  auto at_store = [&](int64_t se, int kvalid, int u, u32x4_t h) __attribute__((always_inline)) {
    const u32x2_t v = {(h[0] | (h[1] << 16)) & at_m01, (h[2] | (h[3] << 16)) & at_m23};
    const bool ok = at_zok && 4 * u + at_c < kvalid;
    const int off = ok ? at_off + u * at_ld8 : 0x7FFFFFF8;
    __builtin_amdgcn_raw_buffer_store_b64(
        v, make_rsrc(p.at + se * BK * p.ldat, (int64_t)kvalid * p.ldat * 2), off, 0, 0);
  };
  // first piece of stage se owned by this tile, (tn - 16 se) mod tiles_n (>= 16: none); the
  // second is at + tiles_n.  In the loop it is stepped, not divided: stage se + 1's is
  // this one minus 16 mod tiles_n.
  auto at_first = [&](int64_t se) -> int {
    const int64_t t = p.tiles_n;
    return (int)((at_tn - (se * 16) % t + t) % t);
  };
  int at_u = 0;
  int at_u_wrap = 0, at_d = 0;
  if (AT) {
    at_u_wrap = at_first(ks0);                   // the stage after the wrap to ks0
    at_d = (int)(16 % p.tiles_n);
  }
  // The main loop's form of at_read / at_store, split into small pieces that go into the
  // issue slots between MFMAs (with one wavefront per SIMD a slot has room for a few
  // instructions only; more stall the MFMA stream).  With kc = 4 u + at_c (at_c < 4),
  // kc >> 3 = u >> 1 and kc & 7 = 4 (u & 1) + at_c, so element e of piece u sits at
  // at_lb[e] + ((u >> 1) << 4 ^ at_sw[e >> 1]) + 8 (u & 1) in the stage (rows at_r + e share
  // (row >> 1) & 7 in pairs).  at_read2 reads elements e0, e0 + 1 of piece u (u < 16) from
  // buffer buf.
  int at_lb[4], at_sw[2];
#pragma unroll
  for (int e = 0; e < 4; ++e) at_lb[e] = (at_r + e) * kRow + at_c * 2;
#pragma unroll
  for (int e = 0; e < 2; ++e) at_sw[e] = (((at_r + 2 * e) >> 1) & 7) << 4;
  auto at_read2 = [&](int buf, int u, int e0, u32x4_t& h) __attribute__((always_inline)) {
    const int xs = (u >> 1) << 4, ad = buf * kStage + ((u & 1) << 3);
    const int x = xs ^ at_sw[e0 >> 1];
    h[e0] = *reinterpret_cast<const uint16_t*>(smem + at_lb[e0] + x + ad);
    h[e0 + 1] = *reinterpret_cast<const uint16_t*>(smem + at_lb[e0 + 1] + x + ad);
  };
  // bytes of a stage's rows of A^T (below 2^31: ldat < 2^24)
  const uint32_t at_sbytes = (uint32_t)(BK * p.ldat * 2);
  auto at_pack = [&](const u32x4_t& h) __attribute__((always_inline)) -> u32x2_t {
    return u32x2_t{(h[0] | (h[1] << 16)) & at_m01, (h[2] | (h[3] << 16)) & at_m23};
  };
  auto at_put = [&](__amdgpu_buffer_rsrc_t r, int u, u32x2_t v) __attribute__((always_inline)) {
    const int off = at_zok && u < 16 ? at_off + u * at_ld8 : 0x7FFFFFF8;
    __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 2);   // non-temporal
  };
  constexpr bool at_two = AT && AT2;             // a second piece per stage is possible
  // One 32-deep slice of TM TN MFMAs from (a, b), with the fragment reads of the next slice (from
  // rst / rkk into ra, rb), one after each MFMA from the first, and, if LOADS, the direct-to-LDS
  // loads [qa, qa + nq) of global stage ls into buffer lbuf, one per CSTEP MFMAs.
  // The scheduling fences keep that interleave.  extra(t) runs after MFMA t (the A^T reads and
  // stores, the packed-B decode, index updates).
  auto slice = [&](auto reads, auto loads, const bf16x8_t* a, const bf16x8_t* b,
                   const char* rst, int rkk, bf16x8_t* ra, bf16x8_t* rb, int ls, int lbuf,
                   int qa, int nq, auto extra) __attribute__((always_inline)) {
    constexpr bool READS = decltype(reads)::value, LOADS = decltype(loads)::value;
    constexpr int NM = TM * TN, NR = TM + TN;
    static_for<NM>([&](auto ti) __attribute__((always_inline)) {
      constexpr int t = decltype(ti)::value;
      // (fragment-major B: by columns, so that B's registers come free one by one, see bf_hook)
      constexpr int i = BF ? t % TM : t / TN, j = BF ? t / TM : t % TN;
      mfma16(acc[i][j], b[j], a[i]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (READS && t < NR) read_one(rst, rkk, t, ra, rb);
      if constexpr (LOADS && t % CSTEP == 1) {
        if (t / CSTEP < nq) dma(ls, lbuf, qa + t / CSTEP);
      }
      extra(t);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // A step computes loop stage s in two slices.  The barrier between them publishes stage s+1
  // (its loads waited) and retires every read of stage s, whose buffer then takes stage s+2's
  // loads: L0 of them in this step's second slice, the rest in the next step's first.  A step
  // knows the global stages of loop stages s and s+1 (e_cur, e_nx1, handed on by the step before)
  // and works out that of s+2 (e_nx2) in a free slot.  LD1 / LD2: loop stages s+1 / s+2 exist (no
  // copies are issued for stages past the end, so the epilogue does not wait for any).  cur: the
  // buffer holding stage s.
  int e_cur = 0, e_nx1 = 0;
  auto step = [&](int s, int s_end, auto last, auto ld1, auto ld2, int cur)
      __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last)::value, LD1 = decltype(ld1)::value;
    constexpr bool LD2 = decltype(ld2)::value;
    constexpr int NM = TM * TN;
    constexpr bool PFS = PF && LD1 && LD2;
    const int nxt = cur ^ 1;
    const char* cs = smem + cur * kStage;
    int e_nx2 = 0;
    auto calc_nx2 = [&]() __attribute__((always_inline)) {
      e_nx2 = gstage(s + 2 < s_end ? s + 2 : s_end - 1);
    };
    if (BQ != 0) calc_nx2();                     // (its registers are loaded early in slice 0)
    // A^T modes: this tile's A^T pieces of the stage (u0 and, with fewer than 16 tile columns,
    // u0 + tiles_n; >= 16: none) are read in slice 0, while the stage is resident, and stored
    // in slice 1, after the barrier; at_u then moves on to stage s+1's piece.
    const int u0 = at_u, u1 = at_u + p.tiles_n;
    u32x4_t v0 = {0, 0, 0, 0}, v1 = {0, 0, 0, 0};
    u32x2_t w0 = {0, 0}, w1 = {0, 0};
    // the main loop's stores cover a full stage (kvalid = BK) of A^T rows
    __amdgpu_buffer_rsrc_t at_rs;
    const char* at_base = nullptr;
    // (slot numbers are for TN = 8, 64 MFMAs a slice; half of them with TN = 4)
    constexpr int H = NM / 32;
    auto at_hook0 = [&](int t) __attribute__((always_inline)) {
      if (!AT) return;
      if (t == 16 * H + 1) at_read2(cur, u0 & 15, 0, v0);
      if (t == 17 * H + 1) at_read2(cur, u0 & 15, 2, v0);
      if (at_two && t == 18 * H + 1) at_read2(cur, u1 & 15, 0, v1);
      if (at_two && t == 19 * H + 1) at_read2(cur, u1 & 15, 2, v1);
      if (t == 22 * H + 1)
        at_base = reinterpret_cast<const char*>(p.at) + (uint64_t)(uint32_t)e_cur * at_sbytes;
      if (t == 24 * H + 1) at_rs = make_rsrc(at_base, (int64_t)at_sbytes);
    };
    auto at_hook1 = [&](int t) __attribute__((always_inline)) {
      if (!AT) return;
      if (t == 18 * H + 1) w0 = at_pack(v0);
      if (t == 20 * H + 1) at_put(at_rs, u0, w0);
      if (at_two && t == 22 * H + 1) w1 = at_pack(v1);
      if (at_two && t == 24 * H + 1) at_put(at_rs, u1, w1);
      if (!LAST && t == 27 * H + 1) {
        int u = e_nx1 == ks0 ? at_u_wrap : at_u - at_d;
        at_u = u < 0 ? u + p.tiles_n : u;
      }
    };
    // Packed B: stage s+2's registers are loaded early in slice 0 (they have until the barrier's
    // wait); stage s+1's second half is decoded into buffer nxt in slice 0, stage s+2's first
    // half into buffer cur in slice 1 (slot g of 24: the g-th decode operation of the half).
    constexpr int kBqHalf = BQ == QF_FMT_NVFP4 ? 24 : BQ == QF_FMT_MXFP4 ? 12 : 23;
    constexpr int BSTEP = NM / 32;               // MFMAs per decode operation
    auto bf_hook = [&](int kk, int t) __attribute__((always_inline)) {
      // after MFMA t = TM j + TM - 1, the last one using fbr[kk][j], that register is loaded with
      // stage s+1's fragment (not in the last step): nearly a whole step before its next use.
      // With all of them at the end of the slice (by rows) and A's copies in slice 0, half a
      // step for either, 2048 x 4096 x 4096 took 85 us, this 77; 8192 x 14336 x 4096 682 / 653
      if (BF && !LAST && t % TM == TM - 1) bf_load(e_nx1, kk, t / TM);
    };
    auto hook0 = [&](int t) __attribute__((always_inline)) {
      if (BQ != 0) {
        if (t == 1) bq_load(e_nx2, bq_nxt);
        const int g = t / BSTEP + kBqHalf;
        if (LD1 && t % BSTEP == 0 && g < kBqOps) bq_op(bq_cur, e_nx1, g, nxt);
      }
      at_hook0(t);
      if (BQ == 0 && t == 15 * H + 1) calc_nx2();
      constexpr int P0 = 17 * H, PS = 2 * H;
      if (PFS && (t == P0 || t == P0 + PS || t == P0 + 2 * PS)) {
        const int q = (t - P0) / PS;
        const int e1 = e_nx2 + (kPfDist - 2), e = e1 >= ks1 ? e1 - klen : e1;
        dma16_buf(rs[q ? 1 : 0], pf_off[q], (uint32_t)e * (uint32_t)kRow, smem + 2 * kStage);
      }
      bf_hook(0, t);
    };
    auto hook1 = [&](int t) __attribute__((always_inline)) {
      if (BQ != 0) {
        const int g = t / BSTEP;
        if (LD2 && t % BSTEP == 0 && g < kBqHalf) bq_op(bq_cur, e_nx2, g, cur);
      }
      at_hook1(t);
      bf_hook(1, t);
    };
    slice(std::true_type{}, std::integral_constant<bool, LD1>{}, fa[0], BF ? fbr[0] : fb[0], cs,
          1, fa[1], fb[1], e_nx1, nxt, L0, NLD - L0, hook0);
    if (BF && !LAST) {
      // A's copies of stage s+1, the last of them after MFMA CSTEP (NLD - 1) + 1 of the previous
      // step's second slice, and everything before them; the B loads issued since, that slice's
      // last ones and this slice's TN, stay in flight (expcnt not waited; lgkmcnt(0): this
      // wavefront's reads of stage s are done before the barrier lets stage s+2's copies
      // overwrite it)
      constexpr int since = TN - (CSTEP * (NLD - 1) + 1) / TM + TN;
      static_assert(since < 16, "the wait's low field");
      __builtin_amdgcn_s_waitcnt(since | (7 << 4) | (0 << 8));
    } else if (PFS) {
      // the three prefetches stay in flight (vmcnt(3), the rest as above)
      __builtin_amdgcn_s_waitcnt(3 | (7 << 4) | (0 << 8));
    } else {
      __builtin_amdgcn_s_waitcnt(0);
    }
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (BQ != 0) bq_cur = bq_nxt;               // complete: the wait above covered its loads
    slice(std::integral_constant<bool, !LAST>{}, std::integral_constant<bool, LD2>{}, fa[1],
          BF ? fbr[BF ? 1 : 0] : fb[1], smem + nxt * kStage, 0, fa[0], fb[0], e_nx2, cur, 0, L0,
          hook1);
    e_cur = e_nx1;
    e_nx1 = e_nx2;
  };

  const int64_t nfull = K / BK;                 // the K tail (dense, second half) follows it
  // (packed or fragment-major B: K is a multiple of BK, checked on the host)
  const int64_t krem = (half == 0 || MODE == kGroupK || BQ != 0 || BF) ? 0 : K % BK;
  const int s0 = ks0, s1 = ks1;
  if (s1 > s0) {
    e_cur = gstage(s0);
    e_nx1 = gstage(s0 + 1 < s1 ? s0 + 1 : s1 - 1);
#pragma unroll
    for (int q = 0; q < NLD; ++q) dma(e_cur, 0, q);
    if (s0 + 1 < s1) {
#pragma unroll
      for (int q = 0; q < L0; ++q) dma(e_nx1, 1, q);
    }
    if (BF) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int j = 0; j < TN; ++j) bf_load(e_cur, kk, j);
    }
  }
  // (the accumulators are cleared while the first copies are under way)
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{};
  acc_settle<true>(acc);
  if (s1 > s0) {
    if (BQ != 0) {
      // stage s0's B decoded now, and the first half of stage s0+1's operations
      BqRegs first;
      bq_load(e_cur, first);
      bq_load(e_nx1, bq_cur);
#pragma unroll
      for (int c = 0; c < 8; ++c) bq_decode(first, e_cur, c, 0);
      if (s0 + 1 < s1) {
        constexpr int kBqHalf = BQ == QF_FMT_NVFP4 ? 24 : BQ == QF_FMT_MXFP4 ? 12 : 23;
#pragma unroll
        for (int u = 0; u < kBqHalf; ++u) bq_op(bq_cur, e_nx1, u, 1);
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_all(smem, 0, fa[0], fb[0]);
    int s = s0;
    if (AT) at_u = at_first(e_cur);
    const std::true_type T{};
    const std::false_type F{};
    // two steps per iteration: with one loop-carried copy of the 256 accumulators the register
    // allocator keeps them in place (a one-step loop body rotates them through other AGPRs at
    // every back edge)
    for (; s + 3 < s1; s += 2) {
      step(s, s1, F, T, T, 0);
      step(s + 1, s1, F, T, T, 1);
    }
    mfma_wait();
    if (s + 2 < s1) {
      step(s, s1, F, T, T, 0);
      mfma_wait();
      ++s;
    }
    if (s + 1 < s1) {
      step(s, s1, F, T, F, (s - s0) & 1);
      mfma_wait();
      ++s;
    }
    step(s, s1, T, F, F, (s - s0) & 1);
    mfma_wait();
  }
  if (krem > 0) {
    // Partial last stage: masked loads through registers into buffer 0.  The wait + barrier
    // retires every earlier read of that buffer.
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
      const int c = (lane & 7) ^ ((4 * (q & 1) + (lane >> 4)) & 7);
      uint4 v = make_uint4(0, 0, 0, 0);
      if (nfull * BK + c * 8 < K)
        v = *reinterpret_cast<const uint4*>(gb[q < TM ? 0 : 1] + nfull * kRow + goff[q]);
      *reinterpret_cast<uint4*>(smem + lds_of(q) + lane * 16) = v;
    }
    __syncthreads();
    if (AT) {                      // the tail stage, same ownership
      for (int u = at_first(nfull); u < 16; u += p.tiles_n)
        at_store(nfull, (int)krem, u, at_read(smem, u));
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      if (kk * 32 >= krem) break;                // uniform: the rest of the stage is zeros
      read_all(smem, kk, fa[0], fb[0]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          mfma16(acc[i][j], fb[0][j], fa[0][i]);
    }
  }

  acc_settle<false>(acc);

  // ---- epilogue: the tile goes through LDS and leaves as whole-row 16-byte stores ----------
  // Each MFMA takes the B fragment as its first operand, so accumulator block (i, j) holds the
  // transposed product: lane l owns columns 4 (l / 16) .. +3 of row l % 16 of the block, written
  // to LDS with one 8-byte (bf16) or 16-byte (FP32) store.
  __syncthreads();                               // every wavefront is done with the operands
  // Destination: the output tile, or (split halves) a dense BM x BN FP32 partial.
  char* Cp = reinterpret_cast<char*>(p.C) + cofs * (C_F32 ? 4 : 2);
  int64_t ldc = p.ldc, em0 = m0, em_end = m_end, en0 = n0, en_end = n_end;
  int vec = p.vec_store;
  if (half >= 0) {
    Cp = reinterpret_cast<char*>(p.part + (int64_t)pidx * BM * BN);
    ldc = BN; em0 = 0; em_end = BM; en0 = 0; en_end = BN; vec = 1;
  }
  const int ec = wn * (16 * TN) + 4 * (lane >> 4);  // this lane's first column in block (*, 0)
  if (!C_F32) {
    // bf16 pairs by the hardware pack (round to nearest even; a NaN result stays a quiet NaN)
    const int er = wm * (16 * TM) + (lane & 15);    // its row in block (0, *)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x4_t& a = acc[i][j];
        *reinterpret_cast<uint2*>(smem + (er + 16 * i) * kPitch16 + (ec + 16 * j) * 2) =
            make_uint2(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
      }
    lds_barrier();
    store_rows16<BM, BN, kPitch16, 256>(smem, Cp, ldc, em0, em_end, en0, en_end, vec);
  } else {
    // FP32 tile in two halves: in half h every wavefront writes its row blocks 4 h .. 4 h + 3, so
    // LDS row q (0..127) holds tile row (q / 64) * 128 + 64 h + q % 64.
    constexpr int HB = TM / 2;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h) lds_barrier();                      // half 0 has been read out of LDS
#pragma unroll
      for (int ii = 0; ii < HB; ++ii)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const f32x4_t& a = acc[HB * h + ii][j];
          const int q = wm * (16 * HB) + ii * 16 + (lane & 15);
          *reinterpret_cast<float4*>(smem + q * kPitch32 + (ec + 16 * j) * 4) =
              make_float4(a[0], a[1], a[2], a[3]);
        }
      lds_barrier();
      store_rows32<BN, kPitch32, 256>(smem, Cp, ldc, em0, em_end, en0, en_end, vec, half < 0,
                                      [&](int q) { return (q >> 6) * 128 + 64 * h + (q & 63); });
    }
  }
}

template <bool C_F32, int MODE, int TM, int TN, int BQ = 0, bool BF = false, bool AT2 = false,
          bool PF = false>
__global__ __launch_bounds__(256, 1) void gemm_nt_kernel(NtArgs p) {
  __shared__ __attribute__((aligned(16))) char smem[nt_smem_bytes(TM, TN, PF)];
  gemm_nt_tile<C_F32, MODE, TM, TN, BQ, BF, AT2, PF>(p, smem);
}

// Grouped rows in tiles of 256 or 128 rows, as launch_grouped_prep has chosen.
__global__ __launch_bounds__(256, 1) void gemm_nt_rows_kernel(NtArgs p) {
  __shared__ __attribute__((aligned(16))) char smem[nt_smem_bytes(8, 8, true)];
  if (p.tile_start[p.E + 1] == 128)
    gemm_nt_tile<false, kGroupRows, 4, 8, 0, false, false, true>(p, smem);
  else
    gemm_nt_tile<false, kGroupRows, 8, 8, 0, false, false, true>(p, smem);
}

// C[tile] = part[2 i] + part[2 i + 1] for the split tiles split_from + i (dense mode, FP32):
// four consecutive columns per lane.  The two halves are added in a fixed order, so the
// result does not depend on which half finished first.
__global__ __launch_bounds__(256) void split_reduce_kernel(NtArgs p) {
  const int i = blockIdx.y;
  const int t = p.split_from + i;
  int64_t m0, n0;
  tile_origin<BM, BN>(p, t, m0, n0);
  const int e = (blockIdx.x * 256 + threadIdx.x) * 4;      // element of the 256 x 256 tile
  const int r = e / BN, c = e % BN;
  const int64_t grow = m0 + r, gcol = n0 + c;
  if (grow >= p.M || gcol >= p.N) return;
  const float4 a = *reinterpret_cast<const float4*>(p.part + (int64_t)(2 * i) * BM * BN + e);
  const float4 b = *reinterpret_cast<const float4*>(p.part + (int64_t)(2 * i + 1) * BM * BN + e);
  const float sum[4] = {a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w};
  float* dst = reinterpret_cast<float*>(p.C) + grow * p.ldc + gcol;
  if (p.vec_store && gcol + 4 <= p.N) {
    *reinterpret_cast<float4*>(dst) = make_float4(sum[0], sum[1], sum[2], sum[3]);
  } else {
    for (int k = 0; k < 4 && gcol + k < p.N; ++k) dst[k] = sum[k];
  }
}

// The loads address a tile with 32-bit byte offsets from its first element: a k-major operand
// spans 256 rows, an mn-major one all K rows.
bool nt_offsets_fit(int64_t K, int64_t lda, int64_t ldb, bool a_mn = false, bool b_mn = false) {
  const int64_t lim = (int64_t)1 << 31;
  const int64_t ra = a_mn ? K + BK : BM, rb = b_mn ? K + BK : BN;
  return K * 2 < lim && ra * lda * 2 < lim && rb * ldb * 2 < lim;
}

int vec_store_ok(const void* C, int64_t ldc, int esize) {
  return (reinterpret_cast<uintptr_t>(C) % 16 == 0) && ((ldc * esize) % 16 == 0);
}

}  // namespace

int64_t compute_units() {
  int dev = 0, ncu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      ncu <= 0)
    return 256;
  return ncu;
}

// With few rows per expert half of a 256-row tile is padding, and the launch chooses between 256 and
// 128 rows on the device (grouped_prep_kernel).  The grouped layer's forward + backward (NVFP4, saved
// operands; E x rows per expert, N x K), us, in 256- / 128-row tiles: 64 x 16, 2048 x 2048 1014 / 973,
// 128 x 64, 3072 x 2048 2961 / 2809, 64 x 96, 2048 x 2048 1065 / 994; no gain from 128 rows per expert
// on (128 x 128, 3072 x 3072 4632 / 4652, 128 x 187 4854 / 4954), where dX writes dY^T instead.
int grouped_tile_rows(int64_t E, int64_t T) { return T <= 96 * E ? 0 : 256; }

size_t gemm_nt_split_bytes(int64_t M, int64_t N) {
  const int64_t tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  return (size_t)(2 * std::min<int64_t>(tiles, kMaxSplitTiles)) * BM * BN * sizeof(float);
}

namespace {

// Launches with at least this many stages prefetch operands into L2 (see the kernel).  What it gains
// depends on the rounds of tiles more than on the stages: panels that an earlier round has read are
// in the last-level cache, those of a single round come from HBM and are waited for.  Measured, us,
// without -> with:
//   one round, 256 x 256 tiles   4096 x 4096 x 2048 54.7 -> 54.2, x 4096 101 -> 96, x 6144 147 -> 141,
//                                x 14336 326 -> 317, x 32768 (FP32) 940 -> 769
//   one round, 256 x 128 tiles   2048 x 4096 x 1024 18.9 -> 20.1, x 2048 41 -> 33, x 4096 79 -> 58,
//                                x 8192 154 -> 116
//   two to four rounds           8192 x 4096 x 4096 193 -> 191, x 14336 660 -> 642; 14336 x 4096 x 6144
//                                516 -> 525, x 14336 1244 -> 1232 (writing A^T 1366 -> 1276)
//   seven rounds                 8192 x 14336 x 4096 647 -> 650, x 8192 1253 -> 1265
// The line at 96 stages takes the long single rounds and costs the many-round launches past it 1 %;
// single rounds of 32 to 95 stages, which would gain most, are below it.
constexpr int64_t kPfMinStages = 96;

// The tile of a dense k-contiguous product: the one whose busiest compute unit copies the fewest
// operand bytes, ceil(tiles / units) (rows + columns), the smaller tile of equals (the figures are
// at the top of qf_gemm_small.hip; 2048 x 4096 x 4096: 84 us in 256 x 256 tiles, 71 in 256 x 128).
// For a bf16 result it depends on M, N and the device alone, so every form of one product (A^T written
// or not, B packed, in fragment order) sums in the same order.  FP32 with a workspace that allows
// halves, which also takes two full stages, is a choice of its own, with its own order of summation.
// halves: FP32 output summed as two K halves; 256 x 256 tiles then run as twice as many half-length
// items plus a pass that adds them (2048 x 2048 x 4096: 63 us, 41 in 128 x 128 tiles that add the
// halves themselves), and the 256 x 128 tile, which does not form halves, is left out.
GemmTile gemm_tile(int64_t M, int64_t N, bool halves = false) {
  static constexpr struct { GemmTile t; int m, n; } kTiles[] = {
      {GemmTile::k256x256, 256, 256}, {GemmTile::k256x128, 256, 128},
      {GemmTile::k128x128, 128, 128}, {GemmTile::k128x64, 128, 64},
      {GemmTile::k64x64, 64, 64},     {GemmTile::k32x32, 32, 32},
      {GemmTile::k16x16, 16, 16}};
  const int64_t cus = compute_units();
  GemmTile best = GemmTile::k256x256;
  int64_t cost = INT64_MAX;
  for (const auto& c : kTiles) {
    const int64_t tiles = ((M + c.m - 1) / c.m) * ((N + c.n - 1) / c.n);
    int64_t v = (tiles + cus - 1) / cus * (c.m + c.n);
    if (halves && c.t == GemmTile::k256x128) continue;
    if (halves && c.t == GemmTile::k256x256) v = tiles > cus ? 0 : v / 2 + 64;
    if (v <= cost) {
      cost = v;
      best = c.t;
    }
  }
  return best;
}

// The dense k-contiguous launch with 32 TN columns per tile.
template <int TN, bool PF>
void launch_form(const NtArgs& a, int c_f32, bool at, dim3 grid, hipStream_t s) {
  const dim3 b(256);
  if (c_f32) hipLaunchKernelGGL((gemm_nt_kernel<true, kDense, 8, TN, 0, false, false, PF>), grid, b, 0, s, a);
  else if (at && a.tiles_n < 16) hipLaunchKernelGGL((gemm_nt_kernel<false, kDenseAT, 8, TN, 0, false, true, PF>), grid, b, 0, s, a);
  else if (at) hipLaunchKernelGGL((gemm_nt_kernel<false, kDenseAT, 8, TN, 0, false, false, PF>), grid, b, 0, s, a);
  else hipLaunchKernelGGL((gemm_nt_kernel<false, kDense, 8, TN, 0, false, false, PF>), grid, b, 0, s, a);
}

// Shared launch of the dense NT GEMM: bf = B in the fragment-major layout (a_mn = b_mn = 0,
// K a multiple of 64).
hipError_t launch_dense(int64_t M, int64_t N, int64_t K, const uint16_t* A, int64_t lda, int a_mn,
                        const uint16_t* B, int64_t ldb, int b_mn, bool bf, void* C, int64_t ldc,
                        int c_f32, float* part, hipStream_t s, uint16_t* at, int64_t ldat) {
  // (a stage's 64 rows of A^T, 128 ldat bytes, stay below 2^31: 32-bit store offsets)
  if (at != nullptr && (c_f32 || a_mn || b_mn || ldat < (M + 7) / 8 * 8 || ldat % 4 != 0 ||
                        ldat >= kGemmAtMaxLd || reinterpret_cast<uintptr_t>(at) % 8 != 0))
    return hipErrorInvalidValue;
  if (bf && (a_mn || b_mn || K % BK != 0 || reinterpret_cast<uintptr_t>(B) % 16 != 0))
    return hipErrorInvalidValue;
  // A last round of 256 x 256 tiles that would leave at least half the CUs idle runs as K-halves
  // instead (FP32 output only; needs a partial buffer and at least two full stages).  The split is
  // decided per XCD: each runs tiles / 8 tiles on cus / 8 CUs.
  const int64_t cus = compute_units();
  const int64_t t256 = ((M + BM - 1) / BM) * ((N + BN - 1) / BN), rem = t256 % cus;
  const bool halves = c_f32 && part != nullptr && t256 % kXcds == 0 && cus % kXcds == 0 &&
                      rem > 0 && 2 * rem <= cus && rem <= kMaxSplitTiles && K / BK >= 2;
  const bool nt = !a_mn && !b_mn;
  const GemmTile tile = nt ? gemm_tile(M, N, halves) : GemmTile::k256x256;
  const bool large = bf || tile == GemmTile::k256x256 || tile == GemmTile::k256x128;
  const int tn = !bf && tile == GemmTile::k256x128 ? 4 : 8;   // 32-column blocks of a tile
  if (at != nullptr && (N == 0 || !large || (N + 32 * tn - 1) / (32 * tn) < 8)) {
    // no tiles, the small kernel, or fewer than 8 tile columns (a tile would own more than two
    // A^T pieces per stage): the transpose kernel writes A^T instead
    if (M > 0 && K > 0) {
      const hipError_t e = launch_transpose_bf16(A, M, K, lda, at, ldat, 1, 0, 0, s);
      if (e != hipSuccess) return e;
    }
    at = nullptr;
  }
  if (M == 0 || N == 0) return hipSuccess;
  if (!nt_offsets_fit(K, lda, bf ? K : ldb, a_mn, b_mn)) return hipErrorInvalidValue;
  NtArgs a{};
  a.A = A; a.B = B; a.C = C; a.lda = lda; a.ldb = ldb; a.ldc = ldc;
  a.M = M; a.N = N; a.K = K;
  a.at = at; a.ldat = ldat;
  a.vec_store = vec_store_ok(C, ldc, c_f32 ? 4 : 2);
  if (halves) a.split_stage = (K / BK) / 2;
  if (!large) return launch_gemm_small(a, tile, c_f32, s);
  const bool pf = K / BK >= kPfMinStages;
  a.norot = tile != GemmTile::k256x256;
  a.tiles_m = (int)((M + BM - 1) / BM);
  a.tiles_n = (int)((N + 32 * tn - 1) / (32 * tn));
  const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n;
  int64_t items = tiles;
  if (halves) {
    a.part = part;
    a.split_from = (int)(tiles - rem);
    a.full_per_xcd = (int)((tiles - rem) / kXcds);
    a.split_per_xcd = (int)(rem / kXcds);
    items = tiles + rem;
  }
  const dim3 grid((unsigned)items), b(256);
  if (a_mn || b_mn) {
    const hipError_t e = launch_gemm_mn_tiles(a, (int)items, a_mn, b_mn, c_f32, s);
    if (e != hipSuccess) return e;
  } else if (bf) {
    if (c_f32) hipLaunchKernelGGL((gemm_nt_kernel<true, kDense, 8, 8, 0, true>), grid, b, 0, s, a);
    else if (at != nullptr) hipLaunchKernelGGL((gemm_nt_kernel<false, kDenseAT, 8, 8, 0, true, true>), grid, b, 0, s, a);
    else hipLaunchKernelGGL((gemm_nt_kernel<false, kDense, 8, 8, 0, true>), grid, b, 0, s, a);
  } else if (tn == 4) {
    if (pf) launch_form<4, true>(a, c_f32, at != nullptr, grid, s);
    else launch_form<4, false>(a, c_f32, at != nullptr, grid, s);
  } else {
    if (pf) launch_form<8, true>(a, c_f32, at != nullptr, grid, s);
    else launch_form<8, false>(a, c_f32, at != nullptr, grid, s);
  }
  if (a.part != nullptr)
    hipLaunchKernelGGL(split_reduce_kernel, dim3(BM * BN / (256 * 4), (unsigned)rem), dim3(256),
                       0, s, a);
  return hipGetLastError();
}

// Row-major bf16 B [N, K] (row stride ld) -> fragment-major (kBfBlock): one lane per 16-byte
// operand; rows past N (to the next multiple of 32) are zeros.
__global__ __launch_bounds__(256) void frag_pack_kernel(const uint16_t* __restrict__ B, int64_t N,
                                                        int64_t K, int64_t ld,
                                                        uint16_t* __restrict__ out,
                                                        int64_t total) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;   // 16-byte operand index
  if (i >= total) return;
  const int64_t blk = i / 64, L = i % 64;
  const int64_t kblocks = K / 16;
  const int64_t nb = blk / kblocks, kb = blk % kblocks;
  const int64_t n = nb * 32 + L % 32, k = kb * 16 + 8 * (L / 32);
  uint4 v = make_uint4(0, 0, 0, 0);
  if (n < N) v = *reinterpret_cast<const uint4*>(B + n * ld + k);
  *reinterpret_cast<uint4*>(out + i * 8) = v;
}

}  // namespace

size_t gemm_frag_bytes(int64_t N, int64_t K) { return (size_t)((N + 31) / 32) * 32 * K * 2; }

hipError_t launch_frag_pack(const uint16_t* B, int64_t N, int64_t K, int64_t ld, uint16_t* out,
                            hipStream_t s) {
  if (N == 0 || K == 0) return hipSuccess;
  if (K % 16 || ld % 8 || reinterpret_cast<uintptr_t>(B) % 16 || reinterpret_cast<uintptr_t>(out) % 16)
    return hipErrorInvalidValue;
  const int64_t total = (N + 31) / 32 * (K / 16) * 64;
  hipLaunchKernelGGL(frag_pack_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, B,
                     N, K, ld, out, total);
  return hipGetLastError();
}

hipError_t launch_gemm_nt(int64_t M, int64_t N, int64_t K, const uint16_t* A, int64_t lda,
                          int a_mn, const uint16_t* B, int64_t ldb, int b_mn, void* C,
                          int64_t ldc, int c_f32, float* part, hipStream_t s, uint16_t* at,
                          int64_t ldat) {
  return launch_dense(M, N, K, A, lda, a_mn, B, ldb, b_mn, false, C, ldc, c_f32, part, s, at,
                      ldat);
}

hipError_t launch_gemm_nt_bf(int64_t M, int64_t N, int64_t K, const uint16_t* A, int64_t lda,
                             const uint16_t* Bf, void* C, int64_t ldc, int c_f32, float* part,
                             hipStream_t s, uint16_t* at, int64_t ldat) {
  return launch_dense(M, N, K, A, lda, 0, Bf, K, 0, true, C, ldc, c_f32, part, s, at, ldat);
}

hipError_t launch_gemm_nt_packed_b(int64_t M, int64_t N, int64_t K, const uint16_t* A,
                                   int64_t lda, int bfmt, const uint8_t* codes,
                                   const uint8_t* scales, const float* S, uint16_t* C,
                                   int64_t ldc, hipStream_t s) {
  if (K % BK != 0 || (bfmt == QF_FMT_Q4K && K % 256 != 0) || codes == nullptr ||
      (bfmt != QF_FMT_Q4K && scales == nullptr) || (bfmt == QF_FMT_NVFP4 && S == nullptr))
    return hipErrorInvalidValue;
  if (M == 0 || N == 0) return hipSuccess;
  if (!nt_offsets_fit(K, lda, K)) return hipErrorInvalidValue;
  NtArgs a{};
  a.A = A; a.B = nullptr; a.C = C; a.lda = lda; a.ldb = K; a.ldc = ldc;
  a.M = M; a.N = N; a.K = K;
  a.bq_codes = codes; a.bq_scales = scales; a.bq_S = S;
  a.vec_store = vec_store_ok(C, ldc, 2);
  a.tiles_m = (int)((M + BM - 1) / BM);
  a.tiles_n = (int)((N + BN - 1) / BN);
  a.norot = gemm_tile(M, N) != GemmTile::k256x256;
  const dim3 grid((unsigned)((int64_t)a.tiles_m * a.tiles_n)), b4(256);
  switch (bfmt) {
    case QF_FMT_NVFP4:
      hipLaunchKernelGGL((gemm_nt_kernel<false, kDense, 8, 8, QF_FMT_NVFP4>), grid, b4, 0, s, a);
      break;
    case QF_FMT_MXFP4:
      hipLaunchKernelGGL((gemm_nt_kernel<false, kDense, 8, 8, QF_FMT_MXFP4>), grid, b4, 0, s, a);
      break;
    case QF_FMT_Q4K:
      hipLaunchKernelGGL((gemm_nt_kernel<false, kDense, 8, 8, QF_FMT_Q4K>), grid, b4, 0, s, a);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_grouped_nt_rows(int64_t E, int64_t T, int64_t N, int64_t K, const int64_t* off,
                                  const int* tile_start, const uint16_t* A, int64_t lda,
                                  const uint16_t* B, int64_t ldb, int64_t bstride,
                                  uint16_t* C, int64_t ldc, hipStream_t s, uint16_t* at,
                                  int64_t ldat, const int* kstart) {
  if (at != nullptr && ((N + BN - 1) / BN < 8 || kstart == nullptr || ldat % 4 != 0 ||
                        ldat >= kGemmAtMaxLd || reinterpret_cast<uintptr_t>(at) % 8 != 0))
    return hipErrorInvalidValue;
  if (T == 0 || N == 0 || E == 0) return hipSuccess;
  const int rows = grouped_tile_rows(E, T);
  if ((at != nullptr && rows != BM) || !nt_offsets_fit(K, lda, ldb)) return hipErrorInvalidValue;
  NtArgs a{};
  a.A = A; a.B = B; a.C = C; a.lda = lda; a.ldb = ldb; a.ldc = ldc; a.bstride = bstride;
  a.M = T; a.N = N; a.K = K; a.off = off; a.tile_start = tile_start; a.E = (int)E;
  a.at = at; a.ldat = ldat; a.kstart = kstart;
  a.vec_store = vec_store_ok(C, ldc, 2);
  a.tiles_n = (int)((N + BN - 1) / BN);
  a.tiles_m = (int)(rows ? (T + rows - 1) / rows + E : (T + 127) / 128 + E);
  const int64_t per = ((int64_t)a.tiles_m * a.tiles_n + kXcds - 1) / kXcds;
  const dim3 grid((unsigned)(kXcds * per));
  if (at != nullptr && a.tiles_n < 16) hipLaunchKernelGGL((gemm_nt_kernel<false, kGroupRowsAT, 8, 8, 0, false, true, true>), grid, dim3(256), 0, s, a);
  else if (at != nullptr) hipLaunchKernelGGL((gemm_nt_kernel<false, kGroupRowsAT, 8, 8, 0, false, false, true>), grid, dim3(256), 0, s, a);
  else if (rows == 0) hipLaunchKernelGGL(gemm_nt_rows_kernel, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((gemm_nt_kernel<false, kGroupRows, 8, 8, 0, false, false, true>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

// Few rows per expert: a weight tile is read about once, and W_hat need not be written and read
// for that.  Forward, us, from W_hat / decoded here (128-row tiles): 64 x 16 rows, 2048 x 2048 NVFP4
// 431 / 342, MXFP4 337 / 244; 128 x 64, 3072 x 2048 1313 / 1021 and 1041 / 739.  (Also at 96 rows per
// expert, 64 x 2048 x 2048, 454 / 380 and 367 / 279; the bound of 64 is from a slower decode.)
// Q4_K's longer decode is not built in.
// Not where few tiles decode one after another on an otherwise idle chip and W_hat comes back out of
// the 256 MB last-level cache, beside W (NVFP4, 48-64 rows, us; tiles, W_hat): 16 x 768 x 2048, 48,
// 50 MB 62 / 75; 8 x 2048 x 2048, 64, 67 MB 71 / 80; 8 x 3072 x 2048, 96, 100 MB 87 / 91.  From 128 MB
// on it pays from 96 tiles on (8 x 3072 x 3072, 151 MB 159 / 127), and from 128 tiles on throughout
// (16 x 2048 x 1024, 67 MB 62 / 60; 32 x 1024 x 1536, 100 MB 83 / 81; 32 x 2048 x 2048, 256 tiles
// 247 / 205, although 256-row tiles may make one round there and 128-row tiles, the only ones that
// decode, two).
bool grouped_packed_b_ok(int fmt, int64_t E, int64_t T, int64_t N, int64_t K) {
  if ((fmt != QF_FMT_NVFP4 && fmt != QF_FMT_MXFP4) || K <= 0 || K % BK != 0 || T > 64 * E ||
      !nt_offsets_fit(K, K, K))
    return false;
  const int64_t tiles = E * ((N + BN - 1) / BN);
  return tiles >= 128 || (tiles >= 96 && E * N * K >= (int64_t)1 << 26);
}

hipError_t launch_grouped_nt_rows_packed_b(int64_t E, int64_t T, int64_t N, int64_t K,
                                           const int64_t* off, const int* tile_start,
                                           const uint16_t* A, int64_t lda, int bfmt,
                                           const uint8_t* codes, const uint8_t* scales,
                                           const float* S, uint16_t* C, int64_t ldc,
                                           hipStream_t s) {
  if (!grouped_packed_b_ok(bfmt, E, T, N, K) || codes == nullptr || scales == nullptr ||
      (bfmt == QF_FMT_NVFP4 && S == nullptr))
    return hipErrorInvalidValue;
  if (T == 0 || N == 0 || E == 0) return hipSuccess;
  if (!nt_offsets_fit(K, lda, K)) return hipErrorInvalidValue;
  NtArgs a{};
  a.A = A; a.B = nullptr; a.C = C; a.lda = lda; a.ldb = K; a.ldc = ldc;
  a.M = T; a.N = N; a.K = K; a.off = off; a.tile_start = tile_start; a.E = (int)E;
  a.bq_codes = codes; a.bq_scales = scales; a.bq_S = S;
  a.vec_store = vec_store_ok(C, ldc, 2);
  a.tiles_n = (int)((N + BN - 1) / BN);
  a.tiles_m = (int)((T + 127) / 128 + E);
  const int64_t per = ((int64_t)a.tiles_m * a.tiles_n + kXcds - 1) / kXcds;
  const dim3 grid((unsigned)(kXcds * per)), b(256);
  if (bfmt == QF_FMT_NVFP4)
    hipLaunchKernelGGL((gemm_nt_kernel<false, kGroupRows, 4, 8, QF_FMT_NVFP4>), grid, b, 0, s, a);
  else
    hipLaunchKernelGGL((gemm_nt_kernel<false, kGroupRows, 4, 8, QF_FMT_MXFP4>), grid, b, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_grouped_nt_k(int64_t E, int64_t M, int64_t N, int64_t Kpad, const int* kstart,
                                const int* order, const uint16_t* A, int64_t lda,
                                const uint16_t* B, int64_t ldb, float* C, int64_t ldc,
                                int64_t cstride, hipStream_t s) {
  if (E == 0 || M == 0 || N == 0) return hipSuccess;
  if (!nt_offsets_fit(Kpad, lda, ldb)) return hipErrorInvalidValue;
  NtArgs a{};
  a.A = A; a.B = B; a.C = C; a.lda = lda; a.ldb = ldb; a.ldc = ldc; a.cstride = cstride;
  a.M = M; a.N = N; a.K = Kpad; a.kstart = kstart; a.order = order; a.E = (int)E;
  a.vec_store = vec_store_ok(C, ldc, 4) && (cstride * 4) % 16 == 0;
  a.tiles_m = (int)((M + BM - 1) / BM);
  a.tiles_n = (int)((N + BN - 1) / BN);
  const int64_t cmax = ((int64_t)a.tiles_m * a.tiles_n + kXcds - 1) / kXcds;
  const dim3 grid((unsigned)(kXcds * E * cmax));
  hipLaunchKernelGGL((gemm_nt_kernel<true, kGroupK, 8, 8, 0, false, false, true>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace qf
