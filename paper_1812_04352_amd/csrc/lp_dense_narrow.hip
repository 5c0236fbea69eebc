// Narrow and double-precision dense residual layers on the matrix cores: fp64
// widths 8, 16 and 32 (v_mfma_f64_16x16x4_f64) and fp32 widths 8 and 16
// (v_mfma_f32_16x16x4_f32).
//
// Forward step (Section 2.2):  v <- v + h_l sigma(K_n v + b_n) (+ g)
// Adjoint step (Section 3.2):  v <- v + h_l K_n^T (sigma'(K_n u^n + b_n) * v) (+ g)
// MGRIT sweeps follow Algorithm 1 (Section 3.1); modes as in lp_internal.h.
//
// A wave owns 16 examples (a tile) per accumulator set. Lane l = 16 g + j holds the
// VQ = Q/4 features g VQ .. g VQ + VQ - 1 of example j, contiguous in memory. The
// contraction runs over slices: slice s takes feature g VQ + s from lane group g,
// which is the B operand as it lies in the registers. The product's rows are
// permuted to match: row i of output block mb is the feature that register r of
// lane group g holds, g VQ + 4 mb + r, with (r, g) = (i / 4, i % 4) in fp64 and
// (i % 4, i / 4) in fp32 (where the two instructions' accumulators keep row i). So
// the result lies as the state does, and steps chain without moving data. At width
// 8 a lane has two features and a block has two useful registers: half of the
// instruction's rows are zero, two instructions per product.
//
// A layer's weights are 2 to 16 values per lane and each is used by one lane of a
// wave only, so they go from L1/L2 straight to registers, a step ahead, without
// LDS and without barriers; a wave runs ET tiles so that they are shared by 16 ET
// examples. The earlier design (one thread per example, weights broadcast from
// LDS) evaluated Q activations and Q^2 products per thread in a row: a serial
// update of 1003 examples at width 16 in fp64 took 8.1 us per adjoint layer and
// 3.2 us per forward layer, 0.6 and 0.5 here; Peaks-shaped sweeps (2048 layers, 5000
// examples, width 8): finest adjoint FC 251 -> 213 us, 4.6 TB/s.
#include <algorithm>
#include <type_traits>

#include "lp_device.h"
#include "lp_internal.h"

namespace lp {
namespace narrow {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int WAVES = 4;  // waves per sweep workgroup

// Where 256 registers suffice, at least two waves per SIMD are asked for: the
// compiler then keeps the accumulators in the vector registers proper instead of
// moving them in and out of the accumulation registers around every product.
#define LP_NARROW_WAVES(Q) __attribute__((amdgpu_waves_per_eu(Q <= 16 ? 2 : 1, 8)))

template <typename T>
struct Mx;
template <>
struct Mx<double> {
  using V = f64x4;
  __device__ static V mul(double a, double b, V c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row_r(int i) { return i >> 2; }
  __device__ static int row_g(int i) { return i & 3; }
};
template <>
struct Mx<float> {
  using V = f32x4;
  __device__ static V mul(float a, float b, V c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row_r(int i) { return i & 3; }
  __device__ static int row_g(int i) { return i >> 2; }
};

template <int Q>
struct Dim {
  static constexpr int VQ = Q / 4;              // features per lane
  static constexpr int NB = Q < 16 ? 1 : Q / 16;  // output blocks
  static constexpr int NR = VQ < 4 ? VQ : 4;      // useful accumulator registers per block
};

// N consecutive elements with vector loads and stores that need element alignment
// only (weights may be views into a flat parameter vector).
template <typename T, int N>
__device__ __forceinline__ void ldv(T (&r)[N], const T* __restrict__ p) {
  constexpr int W = N * (int)sizeof(T) <= 16 ? N : 16 / (int)sizeof(T);
  typedef T Vec __attribute__((ext_vector_type(W), aligned(sizeof(T))));
#pragma unroll
  for (int i = 0; i < N / W; ++i) {
    const Vec x = reinterpret_cast<const Vec*>(p)[i];
#pragma unroll
    for (int k = 0; k < W; ++k) r[i * W + k] = x[k];
  }
}
template <typename T, int N>
__device__ __forceinline__ void stv(T* __restrict__ p, const T (&r)[N]) {
  constexpr int W = N * (int)sizeof(T) <= 16 ? N : 16 / (int)sizeof(T);
  typedef T Vec __attribute__((ext_vector_type(W), aligned(sizeof(T))));
#pragma unroll
  for (int i = 0; i < N / W; ++i) {
    Vec x;
#pragma unroll
    for (int k = 0; k < W; ++k) x[k] = r[i * W + k];
    reinterpret_cast<Vec*>(p)[i] = x;
  }
}

// One layer's operands of a lane: A rows of K_n (forward) or of K_n^T (transposed).
template <typename T, int Q>
struct Wt {
  T a[Dim<Q>::NB][Dim<Q>::VQ];
};
template <typename T, int Q>
__device__ __forceinline__ void ld_fwd(Wt<T, Q>& w, const T* __restrict__ Kn, int lane) {
  constexpr int VQ = Dim<Q>::VQ;
  const int i = lane & 15, f = Mx<T>::row_g(i) * VQ + Mx<T>::row_r(i);
  const bool in = Mx<T>::row_r(i) < Dim<Q>::NR;
#pragma unroll
  for (int mb = 0; mb < Dim<Q>::NB; ++mb) {
    ldv<T, VQ>(w.a[mb], Kn + (in ? f + 4 * mb : 0) * Q + (lane >> 4) * VQ);
    if constexpr (Dim<Q>::NR < 4) {
#pragma unroll
      for (int s = 0; s < VQ; ++s) w.a[mb][s] = in ? w.a[mb][s] : T(0);
    }
  }
}
template <typename T, int Q>
__device__ __forceinline__ void ld_tr(Wt<T, Q>& w, const T* __restrict__ Kn, int lane) {
  constexpr int VQ = Dim<Q>::VQ;
  const int i = lane & 15, f = Mx<T>::row_g(i) * VQ + Mx<T>::row_r(i);
  const bool in = Mx<T>::row_r(i) < Dim<Q>::NR;
#pragma unroll
  for (int mb = 0; mb < Dim<Q>::NB; ++mb)
#pragma unroll
    for (int s = 0; s < VQ; ++s) {
      const T v = Kn[((lane >> 4) * VQ + s) * Q + (in ? f + 4 * mb : 0)];
      w.a[mb][s] = Dim<Q>::NR < 4 && !in ? T(0) : v;
    }
}

// z[0 .. Q/4) = init + A v
template <typename T, int Q>
__device__ __forceinline__ void prod(T* z, const Wt<T, Q>& w, const T (&v)[Q / 4], const T (&init)[Q / 4]) {
  using D = Dim<Q>;
#pragma unroll
  for (int mb = 0; mb < D::NB; ++mb) {
    typename Mx<T>::V acc;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = r < D::NR ? init[4 * mb + (r < D::NR ? r : 0)] : T(0);
#pragma unroll
    for (int s = 0; s < D::VQ; ++s) acc = Mx<T>::mul(w.a[mb][s], v[s], acc);
#pragma unroll
    for (int r = 0; r < D::NR; ++r) z[4 * mb + r] = acc[r];
  }
}

// sigma (or sigma') of a lane's values, one branch on the activation
template <typename T, int N, bool DERIV>
__device__ __forceinline__ void apply(T (&z)[N], int act) {
  if (act == ACT_TANH) {
#pragma unroll
    for (int i = 0; i < N; ++i) z[i] = DERIV ? dact_f<T, ACT_TANH>(z[i]) : act_f<T, ACT_TANH>(z[i]);
  } else if (act == ACT_RELU) {
#pragma unroll
    for (int i = 0; i < N; ++i) z[i] = DERIV ? dact_f<T, ACT_RELU>(z[i]) : act_f<T, ACT_RELU>(z[i]);
  } else if (act == ACT_SMOOTHRELU) {
#pragma unroll
    for (int i = 0; i < N; ++i) z[i] = DERIV ? dact_f<T, ACT_SMOOTHRELU>(z[i]) : act_f<T, ACT_SMOOTHRELU>(z[i]);
  } else if (DERIV) {
#pragma unroll
    for (int i = 0; i < N; ++i) z[i] = T(1);
  }
}

// U^{kc} + E with E = V - U (Algorithm 1, steps 4-5)
template <typename T, int N>
__device__ __forceinline__ void correct(T (&v)[N], const T* cs, const T* vs) {
  T c[N], d[N];
  ldv<T, N>(c, cs);
  ldv<T, N>(d, vs);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = c[i] + (d[i] - c[i]);
}

// Fixed-order workgroup sum of one double per lane; result in thread 0.
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

// The lane's element offset in a [B][Q] row block for tile t of the wave (clamped to
// a valid example past the batch: such lanes load and compute but store nothing).
struct Ex {
  size_t row;
  bool on;
};
template <int Q>
__device__ __forceinline__ Ex example(long tile, int B) {
  const int lane = threadIdx.x & 63;
  const long e = tile * 16 + (lane & 15);
  return {(size_t)(e < B ? e : B - 1) * Q + (size_t)(lane >> 4) * (Q / 4), e < B};
}

// What one step reads, requested a step ahead: the layer's weights and the rows.
template <typename T, int Q, int ET, bool ADJ>
struct Step {
  Wt<T, Q> w;
  T b[Q / 4];
  T u[ADJ ? ET : 1][Q / 4];  // adjoint: the primal state
  T g[ET][Q / 4];            // right-hand side (coarse levels)
};

// ------------------------------------------------------------------ sweeps
// Workgroup (k, y): interval k, tiles of example block y; y is the fast index, so
// workgroups in flight share an interval's weights in L1 and L2.
template <typename T, int Q, int MODE, int ET, bool HASG>
__global__ __launch_bounds__(64 * WAVES) LP_NARROW_WAVES(Q) void k_fwd_sweep(SweepArgs a, int nblk) {
  constexpr int VQ = Q / 4;
  __shared__ double red[WAVES];
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x / nblk, y = blockIdx.x - k * nblk, Nc = gridDim.x / nblk;
  const size_t slice = (size_t)a.B * Q;
  const T* K = static_cast<const T*>(a.K);
  const T* bb = static_cast<const T*>(a.b) + (lane >> 4) * VQ;
  T* X = static_cast<T*>(a.X);
  const T* G = static_cast<const T*>(a.G);
  const T* Cs = static_cast<const T*>(a.Cs);
  const T* Vn = static_cast<const T*>(a.V);
  const int c = a.c, nsteps = MODE == SWEEP_CORRF ? c - 1 : c;
  const T hl = (T)a.hl, hc = (T)a.hc;
  const long kc = (long)k * c;
  Ex ex[ET];
#pragma unroll
  for (int t = 0; t < ET; ++t) ex[t] = example<Q>(((long)y * WAVES + (threadIdx.x >> 6)) * ET + t, a.B);

  using S = Step<T, Q, ET, false>;
  auto fetch = [&](S& s, int j) {
    const size_t n = (size_t)(kc + j) * a.stride;
    ld_fwd<T, Q>(s.w, K + n * (Q * Q), lane);
    ldv<T, VQ>(s.b, bb + n * Q);
    if (HASG) {
#pragma unroll
      for (int t = 0; t < ET; ++t) ldv<T, VQ>(s.g[t], G + (kc + j + 1) * slice + ex[t].row);
    }
  };
  S s0, s1;
  if (nsteps > 0) fetch(s0, 0);
  T v[ET][VQ], coarse[ET][VQ];
#pragma unroll
  for (int t = 0; t < ET; ++t) {
    if (MODE == SWEEP_FC) {
      // a pending coarse-grid correction of the previous cycle is applied on the fly
      if (Vn) correct<T, VQ>(v[t], Cs + (size_t)k * a.cs_stride * slice + ex[t].row, Vn + (size_t)k * slice + ex[t].row);
      else ldv<T, VQ>(v[t], X + kc * slice + ex[t].row);
      if (k == 0 && ex[t].on) stv<T, VQ>(static_cast<T*>(a.S) + ex[t].row, v[t]);
    } else if (MODE == SWEEP_FRES) {
      ldv<T, VQ>(v[t], Cs + (size_t)k * a.cs_stride * slice + ex[t].row);
    } else {
      correct<T, VQ>(v[t], Cs + (size_t)k * a.cs_stride * slice + ex[t].row, Vn + (size_t)k * slice + ex[t].row);
      if (k > 0 && ex[t].on) stv<T, VQ>(X + kc * slice + ex[t].row, v[t]);
    }
  }
  auto step = [&](const S& cur, int j) {
    T s[ET * VQ];
#pragma unroll
    for (int t = 0; t < ET; ++t) prod<T, Q>(s + t * VQ, cur.w, v[t], cur.b);
    apply<T, ET * VQ, false>(s, a.act);
#pragma unroll
    for (int t = 0; t < ET; ++t) {
#pragma unroll
      for (int i = 0; i < VQ; ++i) {
        // coarse step Phi_{l+1} from the same C-point with the same weights
        if (MODE == SWEEP_FRES && j == 0) coarse[t][i] = v[t][i] + hc * s[t * VQ + i];
        v[t][i] = v[t][i] + hl * s[t * VQ + i];
        if (HASG) v[t][i] += cur.g[t][i];
      }
      if (MODE == SWEEP_CORRF && ex[t].on) stv<T, VQ>(X + (kc + j + 1) * slice + ex[t].row, v[t]);
    }
  };
  // two steps at a time, so that the operands in flight change names and not registers
  for (int j = 0; j < nsteps; j += 2) {
    fetch(s1, min(j + 1, nsteps - 1));
    step(s0, j);
    if (j + 1 >= nsteps) break;
    fetch(s0, min(j + 2, nsteps - 1));
    step(s1, j + 1);
  }

  if (MODE == SWEEP_FC) {
#pragma unroll
    for (int t = 0; t < ET; ++t)
      if (ex[t].on) stv<T, VQ>(static_cast<T*>(a.S) + (size_t)(k + 1) * slice + ex[t].row, v[t]);
  } else if (MODE == SWEEP_FRES) {
    double acc = 0.0;
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      T cn[VQ];
      ldv<T, VQ>(cn, Cs + (size_t)(k + 1) * a.cs_stride * slice + ex[t].row);
#pragma unroll
      for (int i = 0; i < VQ; ++i) {
        const T r = v[t][i] - cn[i];
        if (ex[t].on) acc += (double)r * (double)r;
        coarse[t][i] = v[t][i] - coarse[t][i];  // g_{l+1}^{k+1} = f_{k+1} - Phi_{l+1}(C_k)
      }
      if (ex[t].on) {
        stv<T, VQ>(static_cast<T*>(a.Gn) + (size_t)(k + 1) * slice + ex[t].row, coarse[t]);
        if (a.xn_every > 0 && (k + 1) % a.xn_every == 0)
          stv<T, VQ>(static_cast<T*>(a.Xn) + (size_t)(k + 1) * slice + ex[t].row, cn);
        if (k == 0) {
          ldv<T, VQ>(cn, Cs + ex[t].row);
          stv<T, VQ>(static_cast<T*>(a.Xn) + ex[t].row, cn);
        }
      }
    }
    if (a.partial) {
      const double s = wg_sum(acc, red);
      if (threadIdx.x == 0) a.partial[blockIdx.x] = s;
    }
  } else if (k == Nc - 1) {
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      correct<T, VQ>(v[t], Cs + (size_t)Nc * a.cs_stride * slice + ex[t].row, Vn + (size_t)Nc * slice + ex[t].row);
      if (ex[t].on) stv<T, VQ>(X + (size_t)a.Nl * slice + ex[t].row, v[t]);
    }
  }
}

// sigma' of the step's layer, then w = K^T (sigma' * v)
template <typename T, int Q, int MODE, int ET, bool HASG>
__global__ __launch_bounds__(64 * WAVES) LP_NARROW_WAVES(Q) void k_adj_sweep(SweepArgs a, int nblk) {
  constexpr int VQ = Q / 4;
  __shared__ double red[WAVES];
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x / nblk, y = blockIdx.x - k * nblk, Nc = gridDim.x / nblk;
  const size_t slice = (size_t)a.B * Q;
  const T* K = static_cast<const T*>(a.K);
  const T* bb = static_cast<const T*>(a.b) + (lane >> 4) * VQ;
  const T* Uf = static_cast<const T*>(a.Uf);
  T* X = static_cast<T*>(a.X);
  const T* G = static_cast<const T*>(a.G);
  const T* Cs = static_cast<const T*>(a.Cs);
  const T* Vn = static_cast<const T*>(a.V);
  const int c = a.c, nsteps = MODE == SWEEP_CORRF ? c - 1 : c;
  const T hl = (T)a.hl, hc = (T)a.hc;
  const long top = (long)(k + 1) * c;
  Ex ex[ET];
#pragma unroll
  for (int t = 0; t < ET; ++t) ex[t] = example<Q>(((long)y * WAVES + (threadIdx.x >> 6)) * ET + t, a.B);

  using S = Step<T, Q, ET, true>;
  auto fetch = [&](S& s, int j) {
    const long i = top - 1 - j;
    const size_t n = (size_t)i * a.stride;
    ld_fwd<T, Q>(s.w, K + n * (Q * Q), lane);
    ldv<T, VQ>(s.b, bb + n * Q);
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      ldv<T, VQ>(s.u[t], Uf + n * slice + ex[t].row);
      if (HASG) ldv<T, VQ>(s.g[t], G + (size_t)i * slice + ex[t].row);
    }
  };
  S s0, s1;
  if (nsteps > 0) fetch(s0, 0);
  T v[ET][VQ], coarse[ET][VQ];  // FRES: coarse holds C_{k+1} until the last step, then the coarse step
#pragma unroll
  for (int t = 0; t < ET; ++t) {
    if (MODE == SWEEP_FC) {
      if (Vn)
        correct<T, VQ>(v[t], Cs + (size_t)(k + 1) * a.cs_stride * slice + ex[t].row,
                       Vn + (size_t)(k + 1) * slice + ex[t].row);
      else ldv<T, VQ>(v[t], X + top * slice + ex[t].row);
      if (k == Nc - 1 && ex[t].on) stv<T, VQ>(static_cast<T*>(a.S) + (size_t)Nc * slice + ex[t].row, v[t]);
    } else if (MODE == SWEEP_FRES) {
      ldv<T, VQ>(v[t], Cs + (size_t)(k + 1) * a.cs_stride * slice + ex[t].row);
#pragma unroll
      for (int i = 0; i < VQ; ++i) coarse[t][i] = v[t][i];
    } else {
      correct<T, VQ>(v[t], Cs + (size_t)(k + 1) * a.cs_stride * slice + ex[t].row,
                     Vn + (size_t)(k + 1) * slice + ex[t].row);
      if (k + 1 < Nc && ex[t].on) stv<T, VQ>(X + top * slice + ex[t].row, v[t]);
    }
  }
  T zero[VQ];
#pragma unroll
  for (int q = 0; q < VQ; ++q) zero[q] = T(0);
  auto step = [&](const S& cur, const Wt<T, Q>& wt, int j) {
    T d[ET * VQ];
#pragma unroll
    for (int t = 0; t < ET; ++t) prod<T, Q>(d + t * VQ, cur.w, cur.u[t], cur.b);
    apply<T, ET * VQ, true>(d, a.act);
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      T w[VQ], x[VQ];
      if (MODE == SWEEP_FRES && j == c - 1) {
        // coarse adjoint step from the upper C-point, linearised at the same fine state
#pragma unroll
        for (int q = 0; q < VQ; ++q) x[q] = d[t * VQ + q] * coarse[t][q];
        prod<T, Q>(w, wt, x, zero);
#pragma unroll
        for (int q = 0; q < VQ; ++q) coarse[t][q] = coarse[t][q] + hc * w[q];
      }
#pragma unroll
      for (int q = 0; q < VQ; ++q) x[q] = d[t * VQ + q] * v[t][q];
      prod<T, Q>(w, wt, x, zero);
#pragma unroll
      for (int q = 0; q < VQ; ++q) {
        v[t][q] = v[t][q] + hl * w[q];
        if (HASG) v[t][q] += cur.g[t][q];
      }
      if (MODE == SWEEP_CORRF && ex[t].on) stv<T, VQ>(X + (top - 1 - j) * slice + ex[t].row, v[t]);
    }
  };
  // two steps at a time, so that the operands in flight change names and not
  // registers; the transposed operand comes from the lines the forward one brought in
  for (int j = 0; j < nsteps; j += 2) {
    Wt<T, Q> wt;
    ld_tr<T, Q>(wt, K + (size_t)(top - 1 - j) * a.stride * (Q * Q), lane);
    fetch(s1, min(j + 1, nsteps - 1));
    step(s0, wt, j);
    if (j + 1 >= nsteps) break;
    ld_tr<T, Q>(wt, K + (size_t)(top - 2 - j) * a.stride * (Q * Q), lane);
    fetch(s0, min(j + 2, nsteps - 1));
    step(s1, wt, j + 1);
  }

  if (MODE == SWEEP_FC) {
#pragma unroll
    for (int t = 0; t < ET; ++t)
      if (ex[t].on) stv<T, VQ>(static_cast<T*>(a.S) + (size_t)k * slice + ex[t].row, v[t]);
  } else if (MODE == SWEEP_FRES) {
    double acc = 0.0;
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      T ck[VQ];
      ldv<T, VQ>(ck, Cs + (size_t)k * a.cs_stride * slice + ex[t].row);
#pragma unroll
      for (int q = 0; q < VQ; ++q) {
        const T r = v[t][q] - ck[q];
        if (ex[t].on) acc += (double)r * (double)r;
        coarse[t][q] = v[t][q] - coarse[t][q];  // g_{l+1}^k = f_k - Phibar_{l+1}(C_{k+1})
      }
      if (ex[t].on) {
        stv<T, VQ>(static_cast<T*>(a.Gn) + (size_t)k * slice + ex[t].row, coarse[t]);
        if (a.xn_every > 0 && k % a.xn_every == 0)
          stv<T, VQ>(static_cast<T*>(a.Xn) + (size_t)k * slice + ex[t].row, ck);
        if (k == Nc - 1) {
          ldv<T, VQ>(ck, Cs + (size_t)Nc * a.cs_stride * slice + ex[t].row);
          stv<T, VQ>(static_cast<T*>(a.Xn) + (size_t)Nc * slice + ex[t].row, ck);
        }
      }
    }
    if (a.partial) {
      const double s = wg_sum(acc, red);
      if (threadIdx.x == 0) a.partial[blockIdx.x] = s;
    }
  } else if (k == 0) {
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      correct<T, VQ>(v[t], Cs + ex[t].row, Vn + ex[t].row);
      if (ex[t].on) stv<T, VQ>(X + ex[t].row, v[t]);
    }
  }
}

// ------------------------------------------------------------------ serial solves
// One wave per 16 examples through all steps of a level: a chain whose loads must
// be in flight early, so D steps of them are kept in a register ring (indices
// clamped to valid layers and rows, so that every load is issued unconditionally).
template <typename T, int Q>
__global__ __launch_bounds__(64) LP_NARROW_WAVES(Q) void k_fwd_serial(SerialArgs a) {
  constexpr int VQ = Q / 4, D = Q <= 16 ? 4 : 2;
  const int lane = threadIdx.x & 63;
  const Ex ex = example<Q>(blockIdx.x, a.B);
  const size_t slice = (size_t)a.B * Q;
  const T* K = static_cast<const T*>(a.K);
  const T* bb = static_cast<const T*>(a.b) + (lane >> 4) * VQ;
  T* X = static_cast<T*>(a.X);
  const T* G = static_cast<const T*>(a.G);
  const T hl = (T)a.hl;
  using S = Step<T, Q, 1, false>;
  S ring[D];
  auto fetch = [&](S& s, int i) {
    const int ic = min(i, a.Nl - 1);
    const size_t n = (size_t)ic * a.stride;
    ld_fwd<T, Q>(s.w, K + n * (Q * Q), lane);
    ldv<T, VQ>(s.b, bb + n * Q);
    if (G) ldv<T, VQ>(s.g[0], G + (size_t)(ic + 1) * slice + ex.row);
  };
#pragma unroll
  for (int u = 0; u < D; ++u) fetch(ring[u], u);
  T v[VQ];
  ldv<T, VQ>(v, X + ex.row);
  for (int i0 = 0; i0 < a.Nl; i0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int i = i0 + u;
      if (i >= a.Nl) break;
      T s[VQ];
      prod<T, Q>(s, ring[u].w, v, ring[u].b);
      apply<T, VQ, false>(s, a.act);
#pragma unroll
      for (int q = 0; q < VQ; ++q) {
        v[q] = v[q] + hl * s[q];
        if (G) v[q] += ring[u].g[0][q];
      }
      fetch(ring[u], i + D);
      if (ex.on) stv<T, VQ>(X + (size_t)(i + 1) * slice + ex.row, v);
    }
  }
}

template <typename T, int Q>
__global__ __launch_bounds__(64) LP_NARROW_WAVES(Q) void k_adj_serial(SerialArgs a) {
  constexpr int VQ = Q / 4, D = Q <= 16 ? 4 : 2;
  const int lane = threadIdx.x & 63;
  const Ex ex = example<Q>(blockIdx.x, a.B);
  const size_t slice = (size_t)a.B * Q;
  const T* K = static_cast<const T*>(a.K);
  const T* bb = static_cast<const T*>(a.b) + (lane >> 4) * VQ;
  const T* Uf = static_cast<const T*>(a.Uf);
  T* X = static_cast<T*>(a.X);
  const T* G = static_cast<const T*>(a.G);
  const T hl = (T)a.hl;
  using S = Step<T, Q, 1, true>;
  S ring[D];
  Wt<T, Q> wt[D];
  auto fetch = [&](S& s, Wt<T, Q>& w, int j) {
    const int i = max(a.Nl - 1 - j, 0);
    const size_t n = (size_t)i * a.stride;
    ld_fwd<T, Q>(s.w, K + n * (Q * Q), lane);
    ld_tr<T, Q>(w, K + n * (Q * Q), lane);
    ldv<T, VQ>(s.b, bb + n * Q);
    ldv<T, VQ>(s.u[0], Uf + n * slice + ex.row);
    if (G) ldv<T, VQ>(s.g[0], G + (size_t)i * slice + ex.row);
  };
#pragma unroll
  for (int u = 0; u < D; ++u) fetch(ring[u], wt[u], u);
  T v[VQ], zero[VQ];
#pragma unroll
  for (int q = 0; q < VQ; ++q) zero[q] = T(0);
  ldv<T, VQ>(v, X + (size_t)a.Nl * slice + ex.row);
  for (int j0 = 0; j0 < a.Nl; j0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int j = j0 + u;
      if (j >= a.Nl) break;
      T d[VQ], w[VQ];
      prod<T, Q>(d, ring[u].w, ring[u].u[0], ring[u].b);
      apply<T, VQ, true>(d, a.act);
#pragma unroll
      for (int q = 0; q < VQ; ++q) d[q] *= v[q];
      prod<T, Q>(w, wt[u], d, zero);
#pragma unroll
      for (int q = 0; q < VQ; ++q) {
        v[q] = v[q] + hl * w[q];
        if (G) v[q] += ring[u].g[0][q];
      }
      fetch(ring[u], wt[u], j + D);
      if (ex.on) stv<T, VQ>(X + (size_t)(a.Nl - 1 - j) * slice + ex.row, v);
    }
  }
}

// ------------------------------------------------------------------ residuals
// Workgroup (n, y): forward r = Phi_n(U[n]) - U[n+1]; adjoint r = Phibar_n(Lam[n+1])
// - Lam[n]; writes the sum of r^2 over its 64 run examples. A wave takes run tiles with
// one load of the weights, the next tile's rows requested before the current product.
// One tile per wave read the weights for every 16 examples and left a partial per 64:
// 16 layers of 100000 examples, state, us: fp32 width 8 tanh 54, fp64 width 16 ReLU 100;
// 45 and 82 with runs (the vector-ALU kernels: 45 and 90). fp64 width 8 with tanh is
// bound by tanh itself.
template <typename T, int Q, int DIR>
struct ResidRows {
  T u[Q / 4], x[Q / 4], lam[DIR == DIR_ADJ ? Q / 4 : 1];
  Ex ex;
};
template <typename T, int Q, int DIR>
__global__ __launch_bounds__(64 * WAVES) LP_NARROW_WAVES(Q) void k_resid(ResidArgs a, int nblk, int run) {
  constexpr int VQ = Q / 4;
  __shared__ double red[WAVES];
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x / nblk, y = blockIdx.x - n * nblk;
  const size_t slice = (size_t)a.B * Q;
  const T* K = static_cast<const T*>(a.K) + (size_t)n * (Q * Q);
  const T* U = static_cast<const T*>(a.U) + (size_t)n * slice;
  const T* Lm = DIR == DIR_ADJ ? static_cast<const T*>(a.Lam) + (size_t)n * slice : nullptr;
  const T h = (T)a.h;
  using R = ResidRows<T, Q, DIR>;
  auto fetch = [&](R& r, int i) {
    r.ex = example<Q>(((long)y * run + i) * WAVES + (threadIdx.x >> 6), a.B);
    ldv<T, VQ>(r.u, U + r.ex.row);
    if constexpr (DIR == DIR_FWD) {
      ldv<T, VQ>(r.x, U + slice + r.ex.row);
    } else {
      ldv<T, VQ>(r.lam, Lm + slice + r.ex.row);
      ldv<T, VQ>(r.x, Lm + r.ex.row);
    }
  };
  Wt<T, Q> w, wt;
  T b[VQ], zero[VQ];
  ld_fwd<T, Q>(w, K, lane);
  ldv<T, VQ>(b, static_cast<const T*>(a.b) + (size_t)n * Q + (lane >> 4) * VQ);
  if constexpr (DIR == DIR_ADJ) ld_tr<T, Q>(wt, K, lane);
#pragma unroll
  for (int q = 0; q < VQ; ++q) zero[q] = T(0);
  double acc = 0.0;
  auto step = [&](const R& c) {
    T r[VQ], z[VQ];
    prod<T, Q>(z, w, c.u, b);
    apply<T, VQ, DIR == DIR_ADJ>(z, a.act);
    if constexpr (DIR == DIR_FWD) {
#pragma unroll
      for (int q = 0; q < VQ; ++q) r[q] = (c.u[q] + h * z[q]) - c.x[q];
    } else {
#pragma unroll
      for (int q = 0; q < VQ; ++q) z[q] *= c.lam[q];
      prod<T, Q>(r, wt, z, zero);
#pragma unroll
      for (int q = 0; q < VQ; ++q) r[q] = (c.lam[q] + h * r[q]) - c.x[q];
    }
    if (c.ex.on) {
#pragma unroll
      for (int q = 0; q < VQ; ++q) acc += (double)r[q] * (double)r[q];
    }
  };
  // two tiles at a time, so that the rows in flight change names and not registers
  R r0, r1;
  fetch(r0, 0);
  for (int i = 0; i < run; i += 2) {
    if (i + 1 < run) fetch(r1, i + 1);
    step(r0);
    if (i + 1 >= run) break;
    if (i + 2 < run) fetch(r0, i + 2);
    step(r1);
  }
  const double s = wg_sum(acc, red);
  if (threadIdx.x == 0) a.partial[blockIdx.x] = s;
}

// ------------------------------------------------------------------ gradient
// First pass, workgroup (n, chunk): partial[n][chunk] = (sum s u^T, sum s) over the
// chunk's examples, s = sigma'(K_n u + b_n) * lam^{n+1}. Each wave takes tiles of 16
// examples, the next tile's rows requested during the current one; s and u turn
// from [feature slice][example] to [example][feature] through a tile of LDS that is
// the wave's own (no workgroup barrier), and a second product contracts over four
// examples per instruction. At width 8 one instruction takes eight examples: rows
// and columns 0-7 hold the even group of four, 8-15 the odd group, and the two
// diagonal blocks of the result are added. The waves' sums are added in order.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T, int Q>
__global__ __launch_bounds__(64 * WAVES) LP_NARROW_WAVES(Q) void k_grad(GradArgs a) {
  using D = Dim<Q>;
  constexpr int VQ = D::VQ, NB = D::NB, LD = Q + 16 / (int)sizeof(T);
  constexpr int NOUT = Q * Q + Q;
  constexpr int TS = 16 * LD;
  constexpr int SH = 2 * WAVES * TS > NOUT ? 2 * WAVES * TS : NOUT;
  __shared__ __align__(16) T sh[SH];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, j = lane & 15;
  const int n = blockIdx.x, chunk = blockIdx.y;
  const int per_chunk = (((a.B + a.nchunks - 1) / a.nchunks) + 63) / 64 * 64;
  const int e0 = chunk * per_chunk, e1 = min(a.B, e0 + per_chunk);
  const size_t slice = (size_t)a.B * Q;
  const T* U = static_cast<const T*>(a.U) + (size_t)n * slice + g * VQ;
  const T* L = static_cast<const T*>(a.Lam) + (size_t)(n + 1) * slice + g * VQ;
  Wt<T, Q> w;
  T b[VQ];
  ld_fwd<T, Q>(w, static_cast<const T*>(a.K) + (size_t)n * (Q * Q), lane);
  ldv<T, VQ>(b, static_cast<const T*>(a.b) + (size_t)n * Q + g * VQ);
  T* st = sh + wave * 2 * TS;
  T* ut = st + TS;
  typename Mx<T>::V acc[NB][NB];
  T db[VQ];
#pragma unroll
  for (int x = 0; x < NB; ++x)
#pragma unroll
    for (int y = 0; y < NB; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[x][y][r] = T(0);
#pragma unroll
  for (int q = 0; q < VQ; ++q) db[q] = T(0);
  T un[VQ], ln[VQ];
  auto fetch = [&](int base) {  // a valid row of the batch for every lane
    const size_t e = (size_t)min(base + j, a.B - 1) * Q;
    ldv<T, VQ>(un, U + e);
    ldv<T, VQ>(ln, L + e);
  };
  const int first = e0 + wave * 16;
  if (first < e1) fetch(first);
  for (int base = first; base < e1; base += 16 * WAVES) {
    const bool on = base + j < e1;
    T u[VQ], s[VQ];
    {
      T z[VQ];
      prod<T, Q>(z, w, un, b);
      apply<T, VQ, true>(z, a.act);
#pragma unroll
      for (int q = 0; q < VQ; ++q) {
        // examples past the chunk contribute zeros
        u[q] = on ? un[q] : T(0);
        s[q] = on ? z[q] * ln[q] : T(0);
        db[q] += s[q];
      }
    }
    fetch(base + 16 * WAVES);
    stv<T, VQ>(st + j * LD + g * VQ, s);
    stv<T, VQ>(ut + j * LD + g * VQ, u);
    wave_lds_sync();
    if constexpr (Q >= 16) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int er = (4 * c + g) * LD + j;
        T sa[NB], ub[NB];
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          sa[x] = st[er + 16 * x];
          ub[x] = ut[er + 16 * x];
        }
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
          for (int y = 0; y < NB; ++y) acc[x][y] = Mx<T>::mul(sa[x], ub[y], acc[x][y]);
      }
    } else {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int er = (8 * c + 4 * (j >> 3) + g) * LD + (j & 7);
        acc[0][0] = Mx<T>::mul(st[er], ut[er], acc[0][0]);
      }
    }
    wave_lds_sync();
  }
  // db: over the 16 examples of a lane group
#pragma unroll
  for (int q = 0; q < VQ; ++q)
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) db[q] += __shfl_xor(db[q], off, 64);
  __syncthreads();
  // combine the waves in order in one [Q][Q] (+ [Q]) buffer
  for (int wv = 0; wv < WAVES; ++wv) {
    if (wave == wv) {
      if constexpr (Q >= 16) {
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
          for (int y = 0; y < NB; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              // accumulator register r of lane group g holds row 4 r + g (fp64) or 4 g + r (fp32)
              const int i = sizeof(T) == 8 ? 4 * r + g : 4 * g + r, o = (16 * x + i) * Q + 16 * y + j;
              sh[o] = (wv == 0 ? T(0) : sh[o]) + acc[x][y][r];
            }
      } else {
        // rows i < 8 with columns j < 8, then rows i >= 8 with columns j >= 8
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = sizeof(T) == 8 ? 4 * r + g : 4 * g + r, o = (i & 7) * Q + (j & 7);
            if (i >> 3 == half && j >> 3 == half) sh[o] = (wv == 0 && half == 0 ? T(0) : sh[o]) + acc[0][0][r];
          }
          wave_lds_sync();
        }
      }
      if (j == 0) {
#pragma unroll
        for (int q = 0; q < VQ; ++q) sh[Q * Q + g * VQ + q] = (wv == 0 ? T(0) : sh[Q * Q + g * VQ + q]) + db[q];
      }
    }
    __syncthreads();
  }
  T* out = static_cast<T*>(a.partial) + ((size_t)n * a.nchunks + chunk) * NOUT;
  for (int o = threadIdx.x; o < NOUT; o += 64 * WAVES) out[o] = sh[o];
}

// Second pass: sum the chunk partials in chunk order (in fp64) and scale by h.
template <typename T>
__global__ __launch_bounds__(256) void k_grad_final(GradArgs a, int nw, int nbias) {
  const int nout = nw + nbias;
  const size_t o = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (o >= (size_t)a.N * nout) return;
  const size_t n = o / nout, r = o - n * nout;
  const T* p = static_cast<const T*>(a.partial) + n * a.nchunks * nout + r;
  double s = 0.0;
  for (int ch = 0; ch < a.nchunks; ++ch) s += (double)p[(size_t)ch * nout];
  const T v = (T)(s * a.h);
  if (r < (size_t)nw) static_cast<T*>(a.dK)[n * nw + r] = v;
  else static_cast<T*>(a.db)[n * nbias + (r - nw)] = v;
}

// ------------------------------------------------------------------ launchers

template <typename T, int Q, int ET, bool HASG>
hipError_t sweep_et(int dir, const SweepArgs& a, hipStream_t st, int* partials) {
  const long nblk = (a.B + 16L * WAVES * ET - 1) / (16L * WAVES * ET), grid = (a.Nl / a.c) * nblk;
  if (grid > 0x7fffffffL) return hipErrorNotSupported;
  if (partials) *partials = (int)grid;
  const dim3 gd((unsigned)grid);
  const int nb = (int)nblk;
  if (dir == DIR_FWD) {
    if (a.mode == SWEEP_FC) launch(k_fwd_sweep<T, Q, SWEEP_FC, ET, HASG>, gd, 64 * WAVES, 0, st, a, nb);
    else if (a.mode == SWEEP_FRES) launch(k_fwd_sweep<T, Q, SWEEP_FRES, ET, HASG>, gd, 64 * WAVES, 0, st, a, nb);
    else launch(k_fwd_sweep<T, Q, SWEEP_CORRF, ET, HASG>, gd, 64 * WAVES, 0, st, a, nb);
  } else {
    if (a.mode == SWEEP_FC) launch(k_adj_sweep<T, Q, SWEEP_FC, ET, HASG>, gd, 64 * WAVES, 0, st, a, nb);
    else if (a.mode == SWEEP_FRES) launch(k_adj_sweep<T, Q, SWEEP_FRES, ET, HASG>, gd, 64 * WAVES, 0, st, a, nb);
    else launch(k_adj_sweep<T, Q, SWEEP_CORRF, ET, HASG>, gd, 64 * WAVES, 0, st, a, nb);
  }
  return hipGetLastError();
}

// Two tiles per wave once that still leaves eight waves per SIMD on the chip (1024
// SIMDs): the wave's weight loads are then shared by 32 examples. Width 32 in fp64
// keeps one (a second tile's registers halve the resident waves).
template <typename T, int Q>
hipError_t sweep(int dir, const SweepArgs& a, hipStream_t st, int* partials) {
  if constexpr (Q <= 16) {
    if ((long)(a.Nl / a.c) * ((a.B + 31) / 32) >= 8192)
      return a.G ? sweep_et<T, Q, 2, true>(dir, a, st, partials) : sweep_et<T, Q, 2, false>(dir, a, st, partials);
  }
  return a.G ? sweep_et<T, Q, 1, true>(dir, a, st, partials) : sweep_et<T, Q, 1, false>(dir, a, st, partials);
}

template <typename T, int Q>
hipError_t serial(int dir, const SerialArgs& a, hipStream_t st) {
  const dim3 grid((a.B + 15) / 16);
  if (dir == DIR_FWD) launch(k_fwd_serial<T, Q>, grid, 64, 0, st, a);
  else launch(k_adj_serial<T, Q>, grid, 64, 0, st, a);
  return hipGetLastError();
}

// Tiles per wave: as many as leave 8192 workgroups (four rounds of the chip or more), at
// most 16.
template <typename T, int Q>
hipError_t resid(int dir, const ResidArgs& a, hipStream_t st, int* partials) {
  const long tiles = (a.B + 16L * WAVES - 1) / (16L * WAVES);
  const long run = std::clamp<long>(a.N * tiles / 8192, 1, 16), nblk = (tiles + run - 1) / run, grid = a.N * nblk;
  if (grid > 0x7fffffffL) return hipErrorNotSupported;
  if (partials) *partials = (int)grid;
  const dim3 gd((unsigned)grid);
  if (dir == DIR_FWD) launch(k_resid<T, Q, DIR_FWD>, gd, 64 * WAVES, 0, st, a, (int)nblk, (int)run);
  else launch(k_resid<T, Q, DIR_ADJ>, gd, 64 * WAVES, 0, st, a, (int)nblk, (int)run);
  return hipGetLastError();
}

template <typename T, int Q>
hipError_t grad(const GradArgs& a, hipStream_t st) {
  launch(k_grad<T, Q>, dim3(a.N, a.nchunks), 64 * WAVES, 0, st, a);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  const size_t tot = (size_t)a.N * (Q * Q + Q);
  launch(k_grad_final<T>, (unsigned)((tot + 255) / 256), 256, 0, st, a, Q * Q, Q);
  return hipGetLastError();
}

// f(T, width) for the supported combinations
template <typename F>
hipError_t dispatch(int dtype, int q, F&& f) {
  if (dtype == 0) {
    switch (q) {
      case 8: return f(float(), std::integral_constant<int, 8>{});
      case 16: return f(float(), std::integral_constant<int, 16>{});
    }
  } else {
    switch (q) {
      case 8: return f(double(), std::integral_constant<int, 8>{});
      case 16: return f(double(), std::integral_constant<int, 16>{});
      case 32: return f(double(), std::integral_constant<int, 32>{});
    }
  }
  return hipErrorNotSupported;
}

}  // namespace narrow

bool narrow_supported(int dtype, int q) { return q == 8 || q == 16 || (dtype == 1 && q == 32); }

hipError_t narrow_sweep(int dtype, int q, int dir, const SweepArgs& a, hipStream_t st, int* partials) {
  return narrow::dispatch(dtype, q, [&](auto t, auto w) {
    return narrow::sweep<decltype(t), decltype(w)::value>(dir, a, st, partials);
  });
}
hipError_t narrow_serial(int dtype, int q, int dir, const SerialArgs& a, hipStream_t st) {
  return narrow::dispatch(dtype, q, [&](auto t, auto w) {
    return narrow::serial<decltype(t), decltype(w)::value>(dir, a, st);
  });
}
hipError_t narrow_resid(int dtype, int q, int dir, const ResidArgs& a, hipStream_t st, int* partials) {
  return narrow::dispatch(dtype, q, [&](auto t, auto w) {
    return narrow::resid<decltype(t), decltype(w)::value>(dir, a, st, partials);
  });
}
hipError_t narrow_grad(int dtype, int q, const GradArgs& a, hipStream_t st) {
  return narrow::dispatch(dtype, q, [&](auto t, auto w) { return narrow::grad<decltype(t), decltype(w)::value>(a, st); });
}

}  // namespace lp
