// QAD distillation loss for gfx950 (QATFactory Sec. 3.3, Eq. qad-objective): per token row of
// teacher and student logits (bf16 [L, V]), the forward KL of the two softmax distributions,
// its gradient with respect to the student's logits, and the teacher-student top-1 agreement.
//
// Two passes over a row, with a = z log2(e):
//   pass 1  base-2 statistics of both rows around a reference m,
//             S = sum 2^(a - m)                                      (teacher and student)
//             Q = sum 2^(a_T - m_T) (z_T - z_S)                      (teacher-weighted gap)
//           and the first chunk that holds each row's maximum logit.  Then, in natural units,
//             lse_S - lse_T = ln2 (m_S - m_T + log2 (S_S / S_T)),   KL = Q / S_T + lse_S - lse_T
//           (sum_v p_T (log p_T - log p_S) with log p = z - lse).
//   pass 2  grad[v] = scale / S_S (2^(a_S - m_S) - S_S / S_T 2^(a_T - m_T)), i.e.
//           scale (p_S - p_T), written as bf16.
// No log-sum-exp is formed: rounded at its own size (about 20) it would cost each probability and
// the loss 6e-7, most of the error there was (KL rows of 0.1 against FP64 5.5e-6 -> 1.7e-6, of
// 0.005 8e-5 -> 1.5e-5; gradients that are not the nearest bf16 1.6e-3 -> 1.1e-3 of all).
// What bounds it is HBM (6 bytes per logit) and, nearly as much, the vector units: four exponents,
// at a quarter of the rate, and about 20 other operations per logit.  So
//  - a row is read once: of the 16 waves' chunks a compute unit keeps 8 pairs per lane in registers
//    and 4 in LDS (384 KB of the 594 KB of a 151936-logit row pair); only the rest is read again,
//    mostly from L2 and the last-level cache.
//  - a workgroup stays on its unit and walks over rows; a register pair is refilled from the next
//    row as soon as its gradient is out, so loads run on through pass 2 and the row change.  Narrow
//    vocabularies take two 512-lane workgroups a unit, whose passes overlap.
//  - a new reference of a lane's sums is an integer 7 to 8 above the maximum it was made from, and
//    is replaced only when a maximum passes it: few chunks rescale (exactly, by powers of two), no
//    exponential is above 1, and the arguments of those that count are about -8 (rounded to 2^-22);
//    the element of a maximum is looked for once a row, and only where both maxima are in one chunk.
// 4096 x 151936: 916 -> 768 us; 8192 x 32000: 446 -> 328; 2048 x 65536: 221 -> 164 (against one
// workgroup per row reading it twice; keeping alone 0.95 / 1.03 / 0.95 of its time, with the refills
// 0.90 / 0.78 / 0.87).  Each lane folds its 16-byte chunks in a fixed order and the workgroup merges
// the lanes' statistics in a fixed tree, so the results are deterministic.  The gradient goes out with
// non-temporal stores so it does not evict the logits; a lane reads its chunks for the last time
// before it writes their gradient.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qf.h"
#include "qf_codecs.h"
#include "qf_internal.h"

namespace qf {
namespace {

using namespace codec;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kAhead = 7.0f, kAheadPow = 128.0f;    // how far a new reference is ahead; 2^kAhead
constexpr int kNt = 2;                                // buffer operation: non-temporal
constexpr int kKeepLds = 4, kKeepReg = 8;             // chunk pairs a lane keeps for the gradient
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct Stat {   // softmax statistics in base 2 around the reference m
  float m, S, Q;
};

__device__ __forceinline__ float exp2_safe(float d) {   // 2^d with 2^(-inf) = 0
  return __builtin_amdgcn_exp2f(d);
}

// (m1, S1, Q1) + (m2, S2, Q2) -> the larger reference; an empty side (m = -inf) contributes nothing.
__device__ __forceinline__ Stat merge(Stat x, Stat y) {
  const float m = fmaxf(x.m, y.m);
  const float fx = x.m == m ? 1.0f : exp2_safe(x.m - m);
  const float fy = y.m == m ? 1.0f : exp2_safe(y.m - m);
  return Stat{m, x.S * fx + y.S * fy, x.Q * fx + y.Q * fy};
}

struct ArgMax {  // value of a maximum and the first chunk that holds it
  float v;
  int64_t i;
};

struct LaneMax {  // the same within a lane: the number of its chunk
  float v;
  uint32_t i;
};

struct WaveStat {
  Stat st, ss;
  ArgMax at, as;
};

__device__ __forceinline__ ArgMax amax_merge(ArgMax x, ArgMax y) {
  if (y.v > x.v || (y.v == x.v && y.i < x.i)) return y;
  return x;
}

// The 8 bf16 logits of a 16-byte chunk as FP32 (element k in half k % 2 of dword k / 2).
__device__ __forceinline__ void unpack8_f32(uint4 v, float x[8]) {
  const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    x[2 * q] = as_f32(d[q] << 16);
    x[2 * q + 1] = as_f32(d[q] & 0xFFFF0000u);
  }
}

__device__ __forceinline__ float max3(float a, float b, float c) {
  float m;   // fmaxf would first quiet signalling NaNs, one instruction an operand
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(a), "v"(b), "v"(c));
  return m;
}

__device__ __forceinline__ float max8(const float x[8]) {
  const float a = max3(x[0], x[1], x[2]), b = max3(x[3], x[4], x[5]);
  return max3(max3(a, x[6], x[7]), b, b);
}

// First k with x[k] == m (m is the maximum of x, so one exists).
__device__ __forceinline__ int first_eq8(const float x[8], float m) {
  int k0 = 7;
#pragma unroll
  for (int k = 6; k >= 0; --k) k0 = x[k] == m ? k : k0;
  return k0;
}

// Folds a lane's 8-logit chunk number i into its statistics.
__device__ __forceinline__ void fold_chunk(uint4 vt, uint4 vs, uint32_t i, Stat& st, Stat& ss,
                                           LaneMax& at, LaneMax& as) {
  float xt[8], xs[8];
  unpack8_f32(vt, xt);
  unpack8_f32(vs, xs);
  const float mt = max8(xt), ms = max8(xs);
  if (mt > at.v) at = LaneMax{mt, i};
  if (ms > as.v) as = LaneMax{ms, i};
  const float nmt = mt * kLog2e, nms = ms * kLog2e;
  if (nmt > st.m || nms > ss.m) {                     // new references
    const float rt = nmt > st.m ? ceilf(nmt) + kAhead : st.m;
    const float rs = nms > ss.m ? ceilf(nms) + kAhead : ss.m;
    const float ft = st.m == rt ? 1.0f : exp2_safe(st.m - rt);
    const float fs = ss.m == rs ? 1.0f : exp2_safe(ss.m - rs);
    st = Stat{rt, st.S * ft, st.Q * ft};
    ss = Stat{rs, ss.S * fs, 0.0f};
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float et = exp2_safe(__builtin_fmaf(xt[k], kLog2e, -st.m));
    st.S += et;
    st.Q = __builtin_fmaf(et, xt[k] - xs[k], st.Q);
    ss.S += exp2_safe(__builtin_fmaf(xs[k], kLog2e, -ss.m));
  }
}

// The gradient of one chunk, f (2^(a_S - ms) - q 2^(a_T - mt)) with f = scale / S_S and q = S_S / S_T
// (equal rows: exactly zero).  Finite row statistics make every probability finite, so the hardware
// bf16 pack rounds exactly as bf16_rne; rows with non-finite logits keep the bit-level rounding
// (uniform per workgroup).
__device__ __forceinline__ void grad_chunk(uint4 vt, uint4 vs, float mt, float ms, float q, float f,
                                           bool finite, __amdgpu_buffer_rsrc_t out, uint32_t off) {
  float xt[8], xs[8], g[8];
  unpack8_f32(vt, xt);
  unpack8_f32(vs, xs);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float e_t = exp2_safe(__builtin_fmaf(xt[k], kLog2e, -mt));
    const float e_s = exp2_safe(__builtin_fmaf(xs[k], kLog2e, -ms));
    g[k] = f * __builtin_fmaf(-q, e_t, e_s);
  }
  uint32_t o[4];
  if (finite) {
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = bf16x2_rne_nonnan(g[2 * q], g[2 * q + 1]);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = bf16_rne(g[2 * q]) | (bf16_rne(g[2 * q + 1]) << 16);
  }
  const u32x4 ov = {o[0], o[1], o[2], o[3]};
  __builtin_amdgcn_raw_buffer_store_b128(ov, out, (int)off, 0, kNt);
}

// A window of at most n chunks from chunk c of a row on, as a buffer: loads past its end give
// zeros, stores there are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t window(const uint16_t* row, int64_t c,
                                                         int64_t chunks, int n) {
  const int64_t left = chunks - c;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(row + c * 8), (short)0,
                                           left <= 0 ? 0 : (int)(left < n ? left : n) * 16, 0x27000);
}

__device__ __forceinline__ uint4 load_chunk(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// Folds lanes 0 .. N - 1 into lane 0 (N a power of two) by halving offsets.
template <int N>
__device__ __forceinline__ void merge_lanes(int lane, Stat& st, Stat& ss, ArgMax& at, ArgMax& as) {
#pragma unroll
  for (int off = N / 2; off >= 1; off >>= 1) {
    Stat ot{__shfl_down(st.m, off, 64), __shfl_down(st.S, off, 64), __shfl_down(st.Q, off, 64)};
    Stat os{__shfl_down(ss.m, off, 64), __shfl_down(ss.S, off, 64), 0.0f};
    ArgMax oa{__shfl_down(at.v, off, 64), (int64_t)__shfl_down((long long)at.i, off, 64)};
    ArgMax ob{__shfl_down(as.v, off, 64), (int64_t)__shfl_down((long long)as.i, off, 64)};
    if (lane + off < N) {
      st = merge(st, ot);
      ss = merge(ss, os);
      at = amax_merge(at, oa);
      as = amax_merge(as, ob);
    }
  }
}

__device__ __forceinline__ float first_lane(float v) {
  return as_f32((uint32_t)__builtin_amdgcn_readfirstlane((int)__builtin_bit_cast(uint32_t, v)));
}

__device__ __forceinline__ int64_t first_lane(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
  return ((int64_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | lo;
}

// Makes v's registers opaque: its unpacked halves are not carried along beside it.
__device__ __forceinline__ void pin(uint4& v) {
  asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
}

// GRAD: a gradient is written, and the row's chunks are kept for it.
template <int NT, bool GRAD>
__global__ __launch_bounds__(NT, 4) void qad_kl_kernel(
    const uint16_t* __restrict__ zt, int64_t ldt, const uint16_t* __restrict__ zs, int64_t lds_,
    int64_t L, int64_t V, float gscale, float* __restrict__ row_kl, uint16_t* __restrict__ grad,
    int64_t ldg, int32_t* __restrict__ agree) {
  constexpr int NW = NT / 64;
  constexpr int KR = GRAD ? kKeepReg : 0, KL = GRAD ? kKeepLds : 0;
  __shared__ uint4 keep[KL ? KL * 2 * NT : 1];
  __shared__ WaveStat part[2][NW];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t chunks = V >> 3;

  // Lane t owns chunks t, t + NT, t + 2 NT, ... of a row: the first KR pairs stay in registers,
  // the next KL go to LDS (nobody else touches a lane's LDS), the rest is read again for the
  // gradient.  All but the register part moves through two staging pairs.
  uint4 rt[KR ? KR : 1], rs[KR ? KR : 1], vt[2], vs[2];
  constexpr int kStep = NT * 16;                      // bytes from a lane's chunk to its next
  constexpr int kKeep = (KR + KL) * NT;
  uint32_t off = t * 16;
  int head = (int)(chunks < kKeep ? chunks : kKeep);  // chunks of the kept part
  {
#pragma unroll
    for (int j = 0; j < KR; ++j) {
      rt[j] = load_chunk(window(zt + blockIdx.x * ldt, 0, chunks, kKeep), off + j * kStep);
      rs[j] = load_chunk(window(zs + blockIdx.x * lds_, 0, chunks, kKeep), off + j * kStep);
    }
  }
  int par = 0;
  for (int64_t row = blockIdx.x; row < L; row += gridDim.x, par ^= 1) {
    // opaque: conditions and offsets of the unrolled parts are not carried in registers
    if (GRAD) asm volatile("" : "+s"(head), "+v"(off));
    const uint16_t* pt = zt + row * ldt;
    const uint16_t* ps = zs + row * lds_;
    Stat st{-__builtin_huge_valf(), 0.0f, 0.0f};
    Stat ss{-__builtin_huge_valf(), 0.0f, 0.0f};
    LaneMax lt{-__builtin_huge_valf(), 0}, ls{-__builtin_huge_valf(), 0};
    auto stage = [&](int u, int64_t b) __attribute__((always_inline)) {
      vt[u] = load_chunk(window(pt, b, chunks, NT), off);
      vs[u] = load_chunk(window(ps, b, chunks, NT), off);
    };
    stage(0, KR * NT);
    stage(1, (KR + 1) * NT);
#pragma unroll
    for (int j = 0; j < KR; ++j) {
      if (t < head - j * NT) fold_chunk(rt[j], rs[j], j, st, ss, lt, ls);
      __builtin_amdgcn_sched_barrier(0);              // one chunk's temporaries at a time
      pin(rt[j]);
      pin(rs[j]);
    }
#pragma unroll
    for (int j = 0; j < KL; ++j) {
      const int b = (KR + j) * NT, u = j & 1;
      if (t < head - b) {
        keep[2 * j * NT + t] = vt[u];
        keep[(2 * j + 1) * NT + t] = vs[u];
        fold_chunk(vt[u], vs[u], KR + j, st, ss, lt, ls);
      }
      __builtin_amdgcn_sched_barrier(0);
      stage(u, b + 2 * NT);
    }
    static_assert(kKeepLds % 2 == 0, "the staging pairs alternate");
    uint32_t i = KR + KL;
    for (int64_t b = (KR + KL) * NT; b < chunks; b += 2 * NT, i += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (t < chunks - b - u * NT) fold_chunk(vt[u], vs[u], i + u, st, ss, lt, ls);
        __builtin_amdgcn_sched_barrier(0);
        stage(u, b + (u + 2) * NT);
      }
    }

    if (GRAD) {                                       // the part that was not kept, once more
      stage(0, (KR + KL) * NT);
      stage(1, (KR + KL + 1) * NT);
    }
    // a lane that saw nothing above the initial value has no chunk
    auto in_row = [&](LaneMax m) __attribute__((always_inline)) {
      return ArgMax{m.v, m.v == -__builtin_huge_valf() ? INT64_MAX : (int64_t)m.i * NT + t};
    };
    ArgMax at = in_row(lt), as = in_row(ls);
    // workgroup merge in a fixed tree: within each wave by halving offsets, then (every wave for
    // itself) over the waves in the same way.  The rows alternate between two sets of LDS words:
    // a wave writes a set again only after the next row's barrier, so one barrier a row does.
    merge_lanes<64>(lane, st, ss, at, as);
    if (lane == 0) {
      part[par][wv] = WaveStat{st, ss, at, as};
    }
    __syncthreads();
    if (!GRAD && wv) break;                           // (one row a workgroup, its first wave ends it)
    const WaveStat& o = part[par][lane < NW ? lane : 0];
    st = o.st;
    ss = o.ss;
    at = o.at;
    as = o.as;
    merge_lanes<NW>(lane, st, ss, at, as);
    if (t == 0)
      row_kl[row] = st.Q / st.S + ((ss.m - st.m) + __builtin_amdgcn_logf(ss.S / st.S)) * kLn2;
    if (agree) {
      // The maxima's first chunks; where that is one chunk, its owner looks at the elements (before
      // it writes a gradient there).
      const int64_t it = first_lane(at.i), is = first_lane(as.i);
      if (it != is || it >= chunks) {
        if (t == 0) agree[row] = it == is ? 1 : 0;
      } else if (t == (GRAD ? (int)(it & (NT - 1)) : 0)) {
        float xt[8], xs[8];
        unpack8_f32(*reinterpret_cast<const uint4*>(pt + it * 8), xt);
        unpack8_f32(*reinterpret_cast<const uint4*>(ps + it * 8), xs);
        agree[row] = first_eq8(xt, max8(xt)) == first_eq8(xs, max8(xs)) ? 1 : 0;
      }
    }
    if (GRAD) {
      uint16_t* pg = grad + row * ldg;
      // (the references back near the maxima, where the exponents' arguments are smallest; a sum that
      // overflowed, of logits beyond 1e9 all alike, leaves probabilities of zero)
      const bool inf_t = st.S == __builtin_huge_valf(), inf_s = ss.S == __builtin_huge_valf();
      const float mt = first_lane(inf_t ? st.S : st.m - kAhead);
      const float ms = first_lane(inf_s ? ss.S : ss.m - kAhead);
      const float d = inf_s ? 1.0f : ss.S * kAheadPow;
      const float q = first_lane(d / (st.S * kAheadPow)), f = first_lane(gscale / d);
      const bool finite = __builtin_isfinite(mt) && __builtin_isfinite(ms) &&
                          __builtin_isfinite(q) && __builtin_isfinite(f);
      for (int64_t b = (KR + KL) * NT; b < chunks; b += 2 * NT) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          grad_chunk(vt[u], vs[u], mt, ms, q, f, finite, window(pg, b + u * NT, chunks, NT), off);
          __builtin_amdgcn_sched_barrier(0);
          stage(u, b + (u + 2) * NT);
        }
      }
      asm volatile("" : "+s"(head), "+v"(off));
      const auto wg = window(pg, 0, chunks, kKeep);
#pragma unroll
      for (int j = 0; j < KL; ++j) {
        if ((KR + j) * NT < head)                     // uniform
          grad_chunk(keep[2 * j * NT + t], keep[(2 * j + 1) * NT + t], mt, ms, q, f, finite, wg,
                     off + (KR + j) * kStep);
        __builtin_amdgcn_sched_barrier(0);
      }
      // each register pair is refilled from the next row as soon as it is free
      const int64_t next = row + gridDim.x;
      const auto wt = window(zt + next * ldt, 0, next < L ? chunks : 0, kKeep);
      const auto ws = window(zs + next * lds_, 0, next < L ? chunks : 0, kKeep);
#pragma unroll
      for (int j = 0; j < KR; ++j) {
        if (j * NT < head) grad_chunk(rt[j], rs[j], mt, ms, q, f, finite, wg, off + j * kStep);
        __builtin_amdgcn_sched_barrier(0);
        rt[j] = load_chunk(wt, off + j * kStep);
        rs[j] = load_chunk(ws, off + j * kStep);
      }
    }
  }
}

// loss = (1 / L) sum_t row_kl[t] in a fixed order (one workgroup).
__global__ __launch_bounds__(256) void mean_kernel(const float* __restrict__ x, int64_t n,
                                                   float* __restrict__ out) {
  __shared__ float part[256];
  float acc = 0.0f;                                   // x[t], x[t + 256], ... in order,
  int64_t i = threadIdx.x;                            // eight loads in flight per batch
  for (; i + 7 * 256 < n; i += 8 * 256) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x[i + u * 256];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  for (; i < n; i += 256) acc += x[i];
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s >= 1; s >>= 1) {
    if ((int)threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = n > 0 ? part[0] / (float)n : 0.0f;
}

}  // namespace

hipError_t launch_qad_kl(const uint16_t* zt, int64_t ldt, const uint16_t* zs, int64_t lds_,
                         int64_t L, int64_t V, float gscale, float* row_kl, float* loss,
                         uint16_t* grad, int64_t ldg, int32_t* agree, hipStream_t s) {
  if (L > 0) {
    // Two 512-lane workgroups a unit where they keep most of a row (against one of 1024, us: 8192 x
    // 32000 328 / 413, 2048 x 49152 124 / 146, 2048 x 65536 164 / 178, 2048 x 100000 270 / 270, 8192 x
    // 100000 1034 / 1005, 4096 x 151936 845 / 768).  The same with fewer rows than units, where a unit
    // has one of them: 16 x 16384 12.5 / 14.5, 64 x 32000 15.0 / 17.0, 256 x 32000 17.5 / 18.7, 64 x
    // 65536 21.8 / 22.3; and without a gradient, where all four that fit run (the row kernel of one
    // 1024-lane workgroup and a merge by one lane: 4096 x 4096 73.6, 1024 x 32000 43.3, 256 x 32000
    // 15.0): 1024 x 4096 14.6 / 24.7, 1024 x 32000 32.3 / 41.2, 256 x 32000 12.5 / 13.4, 64 x 65536
    // 15.8 / 15.2, 4096 x 65536 187 / 205, 4096 x 151936 418 / 415.
    const bool wide = V > 65536;
    auto* k = wide ? (grad ? &qad_kl_kernel<1024, true> : &qad_kl_kernel<1024, false>)
                   : (grad ? &qad_kl_kernel<512, true> : &qad_kl_kernel<512, false>);
    const int64_t slots = (wide ? 1 : 2) * compute_units();
    hipLaunchKernelGGL(k, dim3((unsigned)(grad && L > slots ? slots : L)), dim3(wide ? 1024 : 512), 0,
                       s, zt, ldt, zs, lds_, L, V, gscale, row_kl, grad, ldg, agree);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (loss) {
    hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(256), 0, s, row_kl, L, loss);
    return hipGetLastError();
  }
  return hipSuccess;
}

}  // namespace qf
