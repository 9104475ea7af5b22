// BF16 MFMA GEMM for gfx950 with operands stored K-as-rows: C[m, n] = sum_k A(m, k) B(n, k), A
// [M][K] or [K][M] (A_MN), B [N][K] or [K][N] (B_MN), at least one of them K-as-rows.
//
// The layer's products run on the k-contiguous kernel (qf_gemm_nt.hip); this form serves the
// plain GEMM's other operand layouts, in place.  256 x 256 block tile, eight wavefronts (two per
// SIMD), each owning a 128 x 64 sub-tile as 4 x 2 v_mfma_f32_32x32x16_bf16 accumulators and
// loading one operand (wavefronts 0-3 A, 4-7 B: 8 direct-to-LDS loads of 1 KB per 64-deep stage,
// double-buffered).  K-as-rows fragments come out of LDS through gfx950's transposing read
// (ds_read_b64_tr_b16).  Stages, barriers, the rotated K walk per XCD, the split of the last
// partial round (FP32 with a workspace) and the epilogue are those of the k-contiguous kernel.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "qf_gemm_common.h"

namespace qf {
namespace {

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int BM = 256, BN = 256;
constexpr int kOpStage = BM * kRow;              // 32 KB: one operand, one stage
constexpr int kStage = 2 * kOpStage;             // 64 KB: A then B
constexpr int kPitch16 = BN * 2 + 16;            // epilogue LDS row pitch, bf16 tile (528 B)
constexpr int kPitch32 = BN * 4 + 32;            // epilogue LDS row pitch, FP32 half tile
constexpr int kSmemEpi = (BM * kPitch16 > 128 * kPitch32) ? BM * kPitch16 : 128 * kPitch32;
constexpr int kSmem = (2 * kStage > kSmemEpi) ? 2 * kStage : kSmemEpi;

// ds_read_b64_tr_b16 (gfx950): transposing 4 x 16-bit LDS read, see the fragment offsets.
__device__ __forceinline__ v4i16 lds_tr16(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4i16*)(__attribute__((address_space(3))) char*)(p));
}

template <bool C_F32, bool A_MN, bool B_MN>
__global__ __launch_bounds__(512, 1) void gemm_mn_kernel(NtArgs p) {
  constexpr int NJ = 2, NLD = 8;
  // stage s+1's loads: L0 in the last slice of step s-1, L1 in slice 0 and L2 in slice 1
  constexpr int L0 = 3, L1 = 3, L2 = NLD - L0 - L1;
  __shared__ __attribute__((aligned(16))) char smem[kSmem];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform (scalar) index
  const int wm = w >> 2, wn = w & 3;
  const int item = remap_xcd(blockIdx.x, gridDim.x);
  int bid = item, half = -1, pidx = 0;
  if (C_F32 && p.part != nullptr) split_item(p, item, bid, half, pidx);
  int64_t m0, n0;
  tile_origin<BM, BN>(p, bid, m0, n0);
  const int64_t m_end = p.M, n_end = p.N, K = p.K;
  int ks0 = 0, ks1 = (int)(K / BK);

  // ---- this lane's loads ----------------------------------------------------------------------
  // Wavefront w loads operand w >> 2, rows (or k-rows) of quarter lw = w & 3: load q lands at LDS
  // offset op * 32 KB + 8 KB lw + 1 KB q.
  // k-major operand ([rows][K], a stage is 256 rows x 128 B): load q covers tile rows
  // R = 64 lw + 8 q .. R + 7, lane l lands at row R + l / 8, slot l % 8 and so fetches logical
  // chunk (l % 8) ^ ((row >> 1) % 8) = (l % 8) ^ ((4 (q % 2) + l / 16) % 8).
  // mn-major operand ([K][rows], a stage is 64 k-rows x 512 B): load q covers k-rows
  // 16 lw + 2 q + {0, 1}; lane l lands at k-row 16 lw + 2 q + l / 32, 16-byte slot l % 32,
  // and fetches logical chunk (l % 32) ^ (4 (k-row % 4)) (chunk c = columns 8c..8c+7).
  const int lw = w & 3, op = w >> 2;
  const bool mn = op ? B_MN : A_MN;              // uniform
  const int64_t ld = op ? p.ldb : p.lda;
  const int64_t r0 = op ? n0 : m0;
  const int64_t rlim = (op ? n_end : m_end) - r0 - 1;   // last valid row (k-major) / column
  const char* gb;
  __amdgpu_buffer_rsrc_t rs;
  int64_t sstride = kRow;                        // bytes from one stage to the next
  uint32_t goff[NLD];
  if (!mn) {
    gb = reinterpret_cast<const char*>((op ? p.B : p.A) + r0 * ld);
    rs = make_rsrc(gb, (rlim * ld + K) * 2);
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
      const int64_t row = lw * 64 + q * 8 + (lane >> 3);
      const int64_t rc = row < rlim ? row : rlim;
      const int c = (lane & 7) ^ ((4 * (q & 1) + (lane >> 4)) & 7);
      goff[q] = (uint32_t)((rc * ld + c * 8) * 2);
    }
  } else {
    gb = reinterpret_cast<const char*>((op ? p.B : p.A) + r0);
    rs = make_rsrc(gb, ((K - 1) * ld + rlim + 1) * 2);
    sstride = (int64_t)BK * ld * 2;
    const int clim = (int)(rlim / 8);            // last chunk holding valid columns
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
      const int kr = lw * 16 + q * 2 + (lane >> 5);
      int c = (lane & 31) ^ (4 * (kr & 3));
      c = c < clim ? c : clim;
      goff[q] = (uint32_t)(((int64_t)kr * ld + c * 8) * 2);
    }
  }
  auto lds_of = [&](int q) { return op * kOpStage + lw * 8192 + q * 1024; };

  // ---- fragment offsets ----------------------------------------------------------------------
  // k-major: slice kk, fragment i at fo[kk] + i * 4096 (32 rows of 128 bytes); fragment rows
  // start 32-aligned, so the swizzle term (row >> 1) & 7 is (lane >> 1) & 7.
  // mn-major: two ds_read_b64_tr_b16 per fragment (k 0-3 and 4-7 of the lane's 8).  Within
  // each group of 16 lanes that instruction hands output lane L element j of source lane
  // 4 j + L / 4 (element L % 4), so source lane 4 j + a points at k-row kb + j, columns
  // c0 + 4 a .. +3: output lane L then holds k-rows kb .. kb+3 of column c0 + L.  Lane l
  // (group g = l / 16) serves MFMA lane rows 16 (g % 2) + L and k-half g / 2; fragment f's base
  // is fo[f], plus (16 kk + 4 h) * 512 bytes for slice kk, half h.
  int foa[4], fob[4];
  {
    const int ra = wm * 128 + (lane & 31), rb = wn * 64 + (lane & 31);
    const int sw = (lane >> 1) & 7;
    const int g = lane >> 4, j = (lane >> 2) & 3, a = lane & 3;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int c = 2 * x + (lane >> 5);
      const int rowj = 8 * (g >> 1) + j;
      if (A_MN) foa[x] = rowj * 512 + ((4 * ((wm * 4 + x) ^ j) + 2 * (g & 1) + (a >> 1)) << 4) + 8 * (a & 1);
      else foa[x] = ra * kRow + ((c ^ sw) << 4);
      if (B_MN) fob[x] = kOpStage + rowj * 512 + ((4 * ((wn * NJ + x) ^ j) + 2 * (g & 1) + (a >> 1)) << 4) + 8 * (a & 1);
      else fob[x] = kOpStage + rb * kRow + ((c ^ sw) << 4);
    }
  }

  f32x16_t acc[4][NJ];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x16_t{};
  bf16x8_t fa[2][4], fb[2][NJ];

  if (half == 1) ks0 = (int)p.split_stage;
  if (half == 0) ks1 = (int)p.split_stage;
  const int klen = ks1 > ks0 ? ks1 - ks0 : 1;
  const int krot = (int)(blockIdx.x % kXcds) * (klen / kXcds);
  auto gstage = [&](int s) __attribute__((always_inline)) -> int {
    const int se = s + krot;
    return se >= ks1 ? se - klen : se;
  };
  const uint32_t sstride32 = (uint32_t)sstride;
  auto dma = [&](int se, int buf, int q) __attribute__((always_inline)) {
    dma16_buf(rs, goff[q], (uint32_t)se * sstride32, smem + buf * kStage + lds_of(q));
  };
  auto frag = [&](const char* st, int kk, int f, bool is_b) __attribute__((always_inline)) -> bf16x8_t {
    const bool mnf = is_b ? B_MN : A_MN;
    if (!mnf) {
      const int* fo = is_b ? fob : foa;
      return *reinterpret_cast<const bf16x8_t*>(st + fo[kk] + f * 4096);
    }
    const char* base = st + (is_b ? fob[f] : foa[f]) + kk * 16 * 512;
    const v4i16 lo = lds_tr16(base);
    const v4i16 hi = lds_tr16(base + 4 * 512);
    const v8i16 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
  };
  // Fragment read r of a slice, in the order the slice's MFMAs consume them: A0, B0, B1, A1..A3.
  auto read_one = [&](const char* st, int kk, int r, bf16x8_t* a, bf16x8_t* b) __attribute__((always_inline)) {
    if (r == 0) a[0] = frag(st, kk, 0, false);
    else if (r <= NJ) b[r - 1] = frag(st, kk, r - 1, true);
    else a[r - NJ] = frag(st, kk, r - NJ, false);
  };
  auto read_all = [&](const char* st, int kk, bf16x8_t* a, bf16x8_t* b) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 4 + NJ; ++r) read_one(st, kk, r, a, b);
  };
  // One 16-deep slice of MFMAs from (a, b), with the fragment reads of the next slice (from
  // rst / rkk into ra, rb) and, if LOADS, loads [qa, qa + nq) of global stage ls into buffer
  // lbuf, one per MFMA.  The scheduling fences keep that interleave.
  auto slice = [&](auto reads, auto loads, const bf16x8_t* a, const bf16x8_t* b,
                   const char* rst, int rkk, bf16x8_t* ra, bf16x8_t* rb, int ls, int lbuf,
                   int qa, int nq) __attribute__((always_inline)) {
    constexpr bool READS = decltype(reads)::value, LOADS = decltype(loads)::value;
    constexpr int NM = 4 * NJ, NR = 4 + NJ;
#pragma unroll
    for (int t = 0; t < NM; ++t) {
      acc[t / NJ][t % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[t % NJ], a[t / NJ],
                                                                    acc[t / NJ][t % NJ], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (READS && t < NR) read_one(rst, rkk, t, ra, rb);
      if (LOADS && t < nq) dma(ls, lbuf, qa + t);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Stage s+1's loads go out L0 in the last slice of step s-1 (right after its barrier freed
  // stage s-1's buffer), L1 in slice 0 and L2 in slice 1 of step s; the barrier before slice 3
  // waits for them.  LD1 / LD2: loop stages s+1 / s+2 exist.  cur: the buffer holding stage s.
  auto step = [&](int s, int s_end, auto last, auto ld1, auto ld2, int cur)
      __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last)::value, LD1 = decltype(ld1)::value;
    constexpr bool LD2 = decltype(ld2)::value;
    const int nxt = cur ^ 1;
    const char* cs = smem + cur * kStage;
    const int e_nx1 = gstage(s + 1 < s_end ? s + 1 : s_end - 1);
    const int e_nx2 = gstage(s + 2 < s_end ? s + 2 : s_end - 1);
    slice(std::true_type{}, std::integral_constant<bool, LD1>{}, fa[0], fb[0], cs, 1, fa[1], fb[1],
          e_nx1, nxt, L0, L1);
    slice(std::true_type{}, std::integral_constant<bool, LD1>{}, fa[1], fb[1], cs, 2, fa[0], fb[0],
          e_nx1, nxt, L0 + L1, L2);
    slice(std::true_type{}, std::false_type{}, fa[0], fb[0], cs, 3, fa[1], fb[1], 0, 0, 0, 0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    slice(std::integral_constant<bool, !LAST>{}, std::integral_constant<bool, LD2>{}, fa[1], fb[1],
          smem + nxt * kStage, 0, fa[0], fb[0], e_nx2, cur, 0, L0);
  };

  const int64_t nfull = K / BK;                 // the K tail (not in a first half) follows it
  const int64_t krem = half == 0 ? 0 : K % BK;
  const int s0 = ks0, s1 = ks1;
  if (s1 > s0) {
    const int e0 = gstage(s0);
#pragma unroll
    for (int q = 0; q < NLD; ++q) dma(e0, 0, q);
    if (s0 + 1 < s1) {
      const int e1 = gstage(s0 + 1);
#pragma unroll
      for (int q = 0; q < L0; ++q) dma(e1, 1, q);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_all(smem, 0, fa[0], fb[0]);
    int s = s0;
    const std::true_type T{};
    const std::false_type F{};
    for (; s + 2 < s1; ++s) step(s, s1, F, T, T, (s - s0) & 1);
    if (s + 1 < s1) {
      step(s, s1, F, T, F, (s - s0) & 1);
      ++s;
    }
    step(s, s1, T, F, F, (s - s0) & 1);
  }
  if (krem > 0) {
    // Partial last stage: masked loads through registers into buffer 0.  The wait + barrier
    // retires every earlier read of that buffer.
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
      bool valid;
      if (!mn) {
        const int c = (lane & 7) ^ ((4 * (q & 1) + (lane >> 4)) & 7);
        valid = nfull * BK + c * 8 < K;
      } else {
        valid = nfull * BK + lw * 16 + q * 2 + (lane >> 5) < K;
      }
      uint4 v = make_uint4(0, 0, 0, 0);
      if (valid) v = *reinterpret_cast<const uint4*>(gb + nfull * sstride + goff[q]);
      *reinterpret_cast<uint4*>(smem + lds_of(q) + lane * 16) = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk * 16 >= krem) break;                // uniform: the rest of the stage is zeros
      read_all(smem, kk, fa[0], fb[0]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[0][j], fa[0][i], acc[i][j], 0, 0, 0);
    }
  }

  // ---- epilogue: the tile goes through LDS and leaves as whole-row 16-byte stores ----------
  // Each MFMA takes the B fragment as its first operand, so accumulator block (i, j) holds the
  // transposed product: element v sits at row lane % 32 of the block and column
  // 8 (v / 4) + 4 (lane / 32) + v % 4, i.e. a lane owns four consecutive columns of one row per
  // group v / 4, written to LDS with one 8-byte (bf16) or 16-byte (FP32) store.
  __syncthreads();                               // every wavefront is done with the operands
  char* Cp = reinterpret_cast<char*>(p.C);
  int64_t ldc = p.ldc, em0 = m0, em_end = m_end, en0 = n0, en_end = n_end;
  int vec = p.vec_store;
  if (half >= 0) {                               // a dense 256 x 256 FP32 partial
    Cp = reinterpret_cast<char*>(p.part + (int64_t)pidx * BM * BN);
    ldc = BN; em0 = 0; em_end = BM; en0 = 0; en_end = BN; vec = 1;
  }
  const int er = wm * 128 + (lane & 31);          // this lane's row in block (0, *)
  const int ec = wn * 64 + 4 * (lane >> 5);       // its first column in block (*, 0), group 0
  if (!C_F32) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x16_t& a = acc[i][j];
          const uint2 o = make_uint2(pack_bf16x2(a[4 * g], a[4 * g + 1]),
                                     pack_bf16x2(a[4 * g + 2], a[4 * g + 3]));
          *reinterpret_cast<uint2*>(smem + (er + 32 * i) * kPitch16 + (ec + 32 * j + 8 * g) * 2) = o;
        }
    lds_barrier();
    store_rows16<BM, BN, kPitch16, 512>(smem, Cp, ldc, em0, em_end, en0, en_end, vec);
  } else {
    // FP32 tile (256 KB) in two halves: in half h every wavefront writes its row blocks 2h and
    // 2h + 1, so LDS row q (0..127) holds tile row (q / 64) * 128 + 64 h + q % 64.
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h) lds_barrier();                      // half 0 has been read out of LDS
#pragma unroll
      for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x16_t& a = acc[2 * h + ii][j];
            const int q = wm * 64 + ii * 32 + (lane & 31);
            *reinterpret_cast<float4*>(smem + q * kPitch32 + (ec + 32 * j + 8 * g) * 4) =
                make_float4(a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]);
          }
      lds_barrier();
      store_rows32<BN, kPitch32, 512>(smem, Cp, ldc, em0, em_end, en0, en_end, vec, half < 0,
                                      [&](int q) { return (q >> 6) * 128 + 64 * h + (q & 63); });
    }
  }
}

}  // namespace

hipError_t launch_gemm_mn_tiles(const NtArgs& a, int items, int a_mn, int b_mn, int c_f32,
                                hipStream_t s) {
  const dim3 grid((unsigned)items), b(512);
  if (c_f32) {
    if (a_mn && b_mn) hipLaunchKernelGGL((gemm_mn_kernel<true, true, true>), grid, b, 0, s, a);
    else if (b_mn) hipLaunchKernelGGL((gemm_mn_kernel<true, false, true>), grid, b, 0, s, a);
    else hipLaunchKernelGGL((gemm_mn_kernel<true, true, false>), grid, b, 0, s, a);
  } else {
    if (a_mn && b_mn) hipLaunchKernelGGL((gemm_mn_kernel<false, true, true>), grid, b, 0, s, a);
    else if (b_mn) hipLaunchKernelGGL((gemm_mn_kernel<false, false, true>), grid, b, 0, s, a);
    else hipLaunchKernelGGL((gemm_mn_kernel<false, true, false>), grid, b, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace qf
