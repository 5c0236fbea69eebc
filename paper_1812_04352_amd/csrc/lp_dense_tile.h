// Tiles of fp32 dense layers of width 32 or 64 on the matrix cores: the staged
// weights, the per-lane layouts of a wave's examples with their products, and the
// activations. Shared by the sweeps and gradient (lp_dense_mfma.hip), the serial
// solves (lp_dense_serial.hip) and the residual norms (lp_dense_resid.hip).
#pragma once

#include <type_traits>

#include "lp_device.h"
#include "lp_internal.h"

namespace lp {
namespace mfma {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// tanh(x) = sign(x) (1 - t) / (1 + t) with t = exp(-2|x|), on the hardware exp2
// and reciprocal; absolute error a few ulp of 1.
__device__ __forceinline__ float tanh_fast(float x) {
  const float t = __builtin_amdgcn_exp2f(-2.885390081777927f * fabsf(x));  // 2 log2(e) |x|
  return copysignf((1.f - t) * __builtin_amdgcn_rcpf(1.f + t), x);
}

template <int Q, int WAVES>
struct Cfg {
  static constexpr int NT = 64 * WAVES;
  static constexpr int MB = Q / 32;               // 32-feature blocks
  static constexpr int LD = Q + 4;                // padded LDS row (floats)
  static constexpr int WSZ = (Q + 1) * LD;        // K rows, then the bias row
  static constexpr int PK = (Q * Q / 4 + NT - 1) / NT;  // float4s of K_n per thread when staging
  static constexpr bool PART = Q * Q / 4 % NT != 0;      // the last float4 slot is not every thread's
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
// four floats in global memory: the caller's arrays may be views into a flat vector, with
// no more than their element's alignment
typedef float f32x4g __attribute__((ext_vector_type(4), aligned(4)));

// One layer's weights in flight between global memory and LDS.
template <int Q, int WAVES>
struct WRegs {
  f32x4 k[Cfg<Q, WAVES>::PK];
  f32x4 b;  // threads < Q/4 carry four bias entries
};

template <int Q, int WAVES>
__device__ __forceinline__ void w_fetch(WRegs<Q, WAVES>& r, const float* __restrict__ K,
                                        const float* __restrict__ b, size_t n) {
  using C = Cfg<Q, WAVES>;
  const f32x4g* Kn = reinterpret_cast<const f32x4g*>(K + n * (size_t)(Q * Q));
#pragma unroll
  for (int p = 0; p < C::PK; ++p) {
    const int idx = threadIdx.x + p * C::NT;
    r.k[p] = (!C::PART || idx < Q * Q / 4) ? (f32x4)Kn[idx] : f32x4{};
  }
  r.b = threadIdx.x < Q / 4 ? (f32x4)reinterpret_cast<const f32x4g*>(b + n * (size_t)Q)[threadIdx.x] : f32x4{};
}

template <int Q, int WAVES>
__device__ __forceinline__ void w_put(float* sh, const WRegs<Q, WAVES>& r) {
  using C = Cfg<Q, WAVES>;
#pragma unroll
  for (int p = 0; p < C::PK; ++p) {
    const int idx = threadIdx.x + p * C::NT;
    if (C::PART && idx >= Q * Q / 4) continue;
    const int el = idx * 4, row = el / Q, col = el - row * Q;
    *reinterpret_cast<f32x4*>(sh + row * C::LD + col) = r.k[p];
  }
  if (threadIdx.x < Q / 4) *reinterpret_cast<f32x4*>(sh + Q * C::LD + threadIdx.x * 4) = r.b;
}

// ------------------------------------------------------------------ layouts
// Per-lane layout of a wave's examples in the accumulators of the two fp32
// matrix-core shapes (lane l):
//   EX = 32, v_mfma_f32_32x32x2_f32: register r of block mb holds feature
//            32mb + 8(r/4) + 4(l/32) + r%4 of example l%32;
//   EX = 16, v_mfma_f32_16x16x4_f32: register r of block mb holds feature
//            16mb + 4(l/16) + r of example l%16.
// In both, the accumulators are the next product's B operand once the A
// operand's contraction index is permuted the same way (k-slice (mb, r) takes
// the feature that register r of block mb holds in each lane group), so chained
// steps never move state between lanes. A wave of the 16-example shape does half
// the work per step with half the latency and needs about two thirds of the
// registers; the sweeps and the serial solve use it, the gradient the other.
// ReLU's sigma' record: one bit per element in element order ([N][B][q], bit f of
// example e's q-bit word, q = 32 or 64), so an example's decisions are one 32- or
// 64-bit word. off is an element offset inside the example's row; the row starts
// at off - off % Q, a multiple of 32 elements, so the word is aligned.
template <int Q>
struct MaskWord {
  static_assert(Q == 32 || Q == 64, "bit records exist for widths 32 and 64");
  using T = typename std::conditional<Q == 64, unsigned long long, uint32_t>::type;
  __device__ static T load(const uint8_t* rec, size_t off) {
    return *reinterpret_cast<const T*>(rec + (off - off % Q) / 8);
  }
  __device__ static void store(uint8_t* rec, size_t off, T w) { *reinterpret_cast<T*>(rec + (off - off % Q) / 8) = w; }
  // 32-bit half i of the word (bits 32 i .. 32 i + 31), shifted right by s: lanes
  // shift once by their own offset and then read bits at constant positions
  __device__ static uint32_t half(T w, int i, int s) { return (uint32_t)(i ? (uint64_t)w >> 32 : w) >> s; }
  // the word from its halves, after an OR over lanes l, l ^ 16, l ^ 32, l ^ 48 (the
  // lanes of one example)
  __device__ static T combine(uint32_t lo, uint32_t hi) {
    lo |= __shfl_xor(lo, 16, 64);
    lo |= __shfl_xor(lo, 32, 64);
    if constexpr (Q == 64) {
      hi |= __shfl_xor(hi, 16, 64);
      hi |= __shfl_xor(hi, 32, 64);
      return ((T)hi << 32) | lo;
    } else {
      return lo;
    }
  }
};
__device__ __forceinline__ float mask_bit(uint32_t h, int b) { return (h >> b) & 1u ? 1.f : 0.f; }

template <int Q, int EX>
struct Lay;

template <int Q>
struct Lay<Q, 32> {
  using V = f32x16;
  static constexpr int NB = Q / 32, NV = 16;

  // p points at the example's row + 4*(lane/32)
  __device__ static void load(V (&v)[NB], const float* __restrict__ p) {
#pragma unroll
    for (int mb = 0; mb < NB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 x = *reinterpret_cast<const f32x4g*>(p + 32 * mb + 8 * g);
#pragma unroll
        for (int t = 0; t < 4; ++t) v[mb][4 * g + t] = x[t];
      }
  }

  __device__ static void store(float* __restrict__ p, const V (&v)[NB]) {
#pragma unroll
    for (int mb = 0; mb < NB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4g*>(p + 32 * mb + 8 * g) =
            f32x4{v[mb][4 * g + 0], v[mb][4 * g + 1], v[mb][4 * g + 2], v[mb][4 * g + 3]};
  }

  // sigma' record of ReLU (bits, MaskWord), off at the lane's element offset
  // e Q + 4 (lane / 32): value (mb, 4 g + t) is feature 32 mb + 8 g + 4 (lane / 32) + t
  __device__ static void load_mask(V (&v)[NB], const uint8_t* __restrict__ rec, size_t off) {
    const auto w = MaskWord<Q>::load(rec, off);
    const int h4 = (int)(off % Q);
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) {
      const uint32_t h = MaskWord<Q>::half(w, mb, h4);
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int t = 0; t < 4; ++t) v[mb][4 * g + t] = mask_bit(h, 8 * g + t);
    }
  }

  // z = K_n v + b_n (W: staged weights, row-major with row pitch LD, bias row last)
  template <int LD>
  __device__ static void prod(V (&z)[NB], const V (&v)[NB], const float* W, int lane) {
    const int h = lane >> 5, i = lane & 31;
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 bb = *reinterpret_cast<const f32x4*>(W + Q * LD + 32 * ob + 8 * g + 4 * h);
#pragma unroll
        for (int t = 0; t < 4; ++t) z[ob][4 * g + t] = bb[t];
      }
      const float* rowp = W + (32 * ob + i) * LD + 4 * h;
#pragma unroll
      for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 a4 = *reinterpret_cast<const f32x4*>(rowp + 32 * ib + 8 * g);
#pragma unroll
          for (int t = 0; t < 4; ++t)
            z[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[t], v[ib][4 * g + t], z[ob], 0, 0, 0);
        }
    }
  }

  // w = K_n^T s (column reads of the staged K_n)
  template <int LD>
  __device__ static void prod_t(V (&w)[NB], const V (&s)[NB], const float* W, int lane) {
    const int h = lane >> 5, i = lane & 31;
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
      w[ob] = 0.f;
      const float* colp = W + 32 * ob + i + 4 * h * LD;
#pragma unroll
      for (int ib = 0; ib < NB; ++ib) {
        // the block's 16 column values are read before its products start
        float a[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) a[r] = colp[(32 * ib + 8 * (r >> 2) + (r & 3)) * LD];
#pragma unroll
        for (int r = 0; r < 16; ++r) w[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[r], s[ib][r], w[ob], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 16, 0);  // LDS reads
        __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);  // then the products
      }
    }
  }
};

template <int Q>
struct Lay<Q, 16> {
  using V = f32x4;
  static constexpr int NB = Q / 16, NV = 4;

  // p points at the example's row + 4*(lane/16)
  __device__ static void load(V (&v)[NB], const float* __restrict__ p) {
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) v[mb] = *reinterpret_cast<const f32x4g*>(p + 16 * mb);
  }

  __device__ static void store(float* __restrict__ p, const V (&v)[NB]) {
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) *reinterpret_cast<f32x4g*>(p + 16 * mb) = v[mb];
  }

  // sigma' record of ReLU (bits, MaskWord), off at the lane's element offset
  // e Q + 4 (lane / 16): value (mb, r) is feature 16 mb + 4 (lane / 16) + r
  __device__ static void load_mask(V (&v)[NB], const uint8_t* __restrict__ rec, size_t off) {
    unpack_mask(v, MaskWord<Q>::load(rec, off), (int)(off % Q));
  }
  // g4 = 4 (lane / 16): value (mb, r) is bit 16 (mb % 2) + r of half mb / 2, shifted by g4
  __device__ static void unpack_mask(V (&v)[NB], typename MaskWord<Q>::T w, int g4) {
#pragma unroll
    for (int i = 0; i < (NB + 1) / 2; ++i) {
      const uint32_t h = MaskWord<Q>::half(w, i, g4);
#pragma unroll
      for (int mb = 2 * i; mb < NB && mb < 2 * i + 2; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[mb][r] = mask_bit(h, 16 * (mb % 2) + r);
    }
  }

  // the four lanes of an example hold disjoint bits of its word: they are combined
  // across lanes (every lane of the wave must call this) and one of them stores it
  __device__ static void store_mask(uint8_t* __restrict__ rec, size_t off, const V (&v)[NB], bool on) {
    const int g4 = (int)(off % Q);
    uint32_t h[2] = {0u, 0u};
#pragma unroll
    for (int mb = 0; mb < NB; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) h[mb / 2] |= (v[mb][r] != 0.f ? 1u : 0u) << (16 * (mb % 2) + r);
    const auto w = MaskWord<Q>::combine(h[0] << g4, h[1] << g4);
    if (on && g4 == 0) MaskWord<Q>::store(rec, off, w);
  }

  // z = K_n v + b_n: A operand of slice (ib, r) in lane l is K[16ob + l%16][16ib + 4(l/16) + r].
  // At width 64 (DB) the A operands (and bias) of output block ob + 1 are read
  // from LDS while block ob's products run, so the products do not wait on LDS
  // latency; the extra registers are what DB = false saves.
  template <int LD, bool DB = true>
  __device__ static void prod(V (&z)[NB], const V (&v)[NB], const float* W, int lane) {
    const int g = lane >> 4, i = lane & 15;
    if constexpr (NB < 4 || !DB) {
      // width 32: two blocks, few registers to spare (up to eight waves per SIMD)
#pragma unroll
      for (int ob = 0; ob < NB; ++ob) {
        z[ob] = *reinterpret_cast<const f32x4*>(W + Q * LD + 16 * ob + 4 * g);
        const float* rowp = W + (16 * ob + i) * LD + 4 * g;
#pragma unroll
        for (int ib = 0; ib < NB; ++ib) {
          const f32x4 a4 = *reinterpret_cast<const f32x4*>(rowp + 16 * ib);
#pragma unroll
          for (int r = 0; r < 4; ++r) z[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[r], v[ib][r], z[ob], 0, 0, 0);
        }
      }
      return;
    }
    f32x4 A[2][NB], bz[2];
    auto rd = [&](int buf, int ob) {
      bz[buf] = *reinterpret_cast<const f32x4*>(W + Q * LD + 16 * ob + 4 * g);
      const float* rowp = W + (16 * ob + i) * LD + 4 * g;
#pragma unroll
      for (int ib = 0; ib < NB; ++ib) A[buf][ib] = *reinterpret_cast<const f32x4*>(rowp + 16 * ib);
    };
    rd(0, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, NB + 1, 0);  // block 0's LDS reads
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
      const int cb = ob & 1;
      if (ob + 1 < NB) rd(cb ^ 1, ob + 1);
      z[ob] = bz[cb];
#pragma unroll
      for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int r = 0; r < 4; ++r) z[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[cb][ib][r], v[ib][r], z[ob], 0, 0, 0);
      if (ob + 1 < NB) __builtin_amdgcn_sched_group_barrier(0x100, NB + 1, 0);  // next block's LDS reads
      __builtin_amdgcn_sched_group_barrier(0x008, 4 * NB, 0);                 // then this block's products
    }
  }

  // w = K_n^T s: A operand of slice (ib, r) in lane l is K[16ib + 4(l/16) + r][16ob + l%16]
  // (column reads of the staged K_n), double-buffered across output blocks as in prod.
  template <int LD, bool DB = true>
  __device__ static void prod_t(V (&w)[NB], const V (&s)[NB], const float* W, int lane) {
    const int g = lane >> 4, i = lane & 15;
    if constexpr (NB < 4 || !DB) {
#pragma unroll
      for (int ob = 0; ob < NB; ++ob) {
        w[ob] = 0.f;
        const float* colp = W + 16 * ob + i + 4 * g * LD;
        float a[NB][4];
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
          for (int r = 0; r < 4; ++r) a[ib][r] = colp[(16 * ib + r) * LD];
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
          for (int r = 0; r < 4; ++r) w[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ib][r], s[ib][r], w[ob], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 4 * NB, 0);  // LDS reads
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * NB, 0);  // then the products
      }
      return;
    }
    float A[2][NB][4];
    auto rd = [&](int buf, int ob) {
      const float* colp = W + 16 * ob + i + 4 * g * LD;
#pragma unroll
      for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int r = 0; r < 4; ++r) A[buf][ib][r] = colp[(16 * ib + r) * LD];
    };
    rd(0, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 4 * NB, 0);  // block 0's LDS reads
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
      const int cb = ob & 1;
      if (ob + 1 < NB) rd(cb ^ 1, ob + 1);
      w[ob] = 0.f;
#pragma unroll
      for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int r = 0; r < 4; ++r) w[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[cb][ib][r], s[ib][r], w[ob], 0, 0, 0);
      if (ob + 1 < NB) __builtin_amdgcn_sched_group_barrier(0x100, 4 * NB, 0);  // next block's LDS reads
      __builtin_amdgcn_sched_group_barrier(0x008, 4 * NB, 0);                 // then this block's products
    }
  }
};

template <typename V, int NB>
__device__ __forceinline__ void add_to(V (&v)[NB], const V (&t)[NB]) {
#pragma unroll
  for (int mb = 0; mb < NB; ++mb) v[mb] += t[mb];
}

// sigma (deriv = false) or sigma' (deriv = true) of every value, one branch on the
// activation for the whole array
template <typename V, int NB, int NV>
__device__ __forceinline__ void apply(V (&z)[NB], int act, bool deriv) {
  switch (act) {
    case ACT_TANH:
#pragma unroll
      for (int mb = 0; mb < NB; ++mb)
#pragma unroll
        for (int r = 0; r < NV; ++r) {
          const float t = tanh_fast(z[mb][r]);
          z[mb][r] = deriv ? 1.f - t * t : t;
        }
      break;
    case ACT_RELU:
#pragma unroll
      for (int mb = 0; mb < NB; ++mb)
#pragma unroll
        for (int r = 0; r < NV; ++r)
          z[mb][r] = deriv ? (z[mb][r] > 0.f ? 1.f : 0.f) : (z[mb][r] > 0.f ? z[mb][r] : 0.f);
      break;
    case ACT_SMOOTHRELU:
#pragma unroll
      for (int mb = 0; mb < NB; ++mb)
#pragma unroll
        for (int r = 0; r < NV; ++r)
          z[mb][r] = deriv ? dact_f<float, ACT_SMOOTHRELU>(z[mb][r]) : act_f<float, ACT_SMOOTHRELU>(z[mb][r]);
      break;
    default:
      if (deriv) {
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) z[mb] = 1.f;
      }
      break;
  }
}

// v = c + (v' - c) (Algorithm 1, the coarse-grid correction of a C-point)
template <typename Lt>
__device__ __forceinline__ void correct(typename Lt::V (&v)[Lt::NB], const float* cs, const float* vs) {
  typename Lt::V cv[Lt::NB], vv[Lt::NB];
  Lt::load(cv, cs);
  Lt::load(vv, vs);
#pragma unroll
  for (int mb = 0; mb < Lt::NB; ++mb) v[mb] = cv[mb] + (vv[mb] - cv[mb]);
}

// Sum of squares of (a - b) over the lane's values, in fp64.
template <typename V, int NB, int NV>
__device__ __forceinline__ double sq_diff(const V (&a)[NB], const V (&b)[NB]) {
  double acc = 0.0;
#pragma unroll
  for (int mb = 0; mb < NB; ++mb)
#pragma unroll
    for (int r = 0; r < NV; ++r) {
      const float d = a[mb][r] - b[mb][r];
      acc += (double)d * (double)d;
    }
  return acc;
}

// The sigma' record at element offset off: bits for ReLU (MaskWord), fp32 otherwise.
template <typename Lt>
__device__ __forceinline__ void load_dsig(typename Lt::V (&d)[Lt::NB], const void* rec, size_t off, int act) {
  if (act == ACT_RELU) Lt::load_mask(d, static_cast<const uint8_t*>(rec), off);
  else Lt::load(d, static_cast<const float*>(rec) + off);
}

// on: whether the lane's example exists; every lane of the wave calls this (the
// ReLU bits of an example are gathered across its lanes)
template <typename Lt>
__device__ __forceinline__ void store_dsig(void* rec, size_t off, int act, const typename Lt::V (&d)[Lt::NB], bool on) {
  if (act == ACT_RELU) Lt::store_mask(static_cast<uint8_t*>(rec), off, d, on);
  else if (on) Lt::store(static_cast<float*>(rec) + off, d);
}

// A sigma' record row as loaded (16-example lanes): the example's word of ReLU's
// decision bits (MaskWord) or the fp32 values of the smooth activations.
template <typename Lt, bool BITS>
struct RecRow;
template <typename Lt>
struct RecRow<Lt, true> {
  static constexpr int Q = 16 * Lt::NB;
  typename MaskWord<Q>::T w;
  __device__ void load(const void* rec, size_t off) { w = MaskWord<Q>::load(static_cast<const uint8_t*>(rec), off); }
  __device__ void get(typename Lt::V (&d)[Lt::NB]) const { Lt::unpack_mask(d, w, 4 * ((threadIdx.x & 63) >> 4)); }
};
template <typename Lt>
struct RecRow<Lt, false> {
  typename Lt::V v[Lt::NB];
  __device__ void load(const void* rec, size_t off) { Lt::load(v, static_cast<const float*>(rec) + off); }
  __device__ void get(typename Lt::V (&d)[Lt::NB]) const {
#pragma unroll
    for (int mb = 0; mb < Lt::NB; ++mb) d[mb] = v[mb];
  }
};

// Fixed-order workgroup sum of one double per lane; result in thread 0.
template <int WAVES>
__device__ __forceinline__ double wg_sum(double v, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < WAVES; ++w) s += red[w];
  return s;
}

}  // namespace mfma
}  // namespace lp
