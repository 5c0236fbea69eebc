// Dense fp32 residual layers of width 32 or 64 on the matrix cores (gfx950
// v_mfma_f32_16x16x4_f32 for the sweeps,
// v_mfma_f32_32x32x2_f32 for the gradient).
//
// One wave owns EX examples (16 or 32) for all steps of an interval. The layer
// product z = K_n v is a (q x q) x (q x EX) contraction: M = output feature,
// N = example, K = input feature. Its accumulator layout (see Lay below) is also
// a valid B-operand layout for the next step once the contraction index is
// permuted the same way in the A operand, so chained steps never move the state
// between lanes. K_n and b_n are staged in LDS (row-major, padded rows,
// double-buffered: the next layer is fetched into registers while the current
// step runs); the bias initialises the accumulators.
//
// Forward step (Section 2.2):  v <- v + h_l sigma(K_n v + b_n) (+ g)
// Adjoint step (Section 3.2):  v <- v + h_l K_n^T (sigma'(K_n u^n + b_n) * v) (+ g);
//   the transposed product reads K_n column-wise from the same LDS copy.
// Sweep modes follow Algorithm 1 exactly as the VALU kernels do (lp_dense_impl.h).
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "lp_dense_tile.h"

namespace lp {
namespace mfma {

// ------------------------------------------------------------------ forward
// Interval k = blockIdx.y, examples of blockIdx.x.
// Consecutive workgroups share an interval, so the round-robin dispatch over the
// 8 XCDs gives each XCD every interval's weights once, in order, and its L2 only
// has to hold the few intervals in flight (with the interval as the fast index,
// an XCD received all tiles of every 8th interval and its weights overflowed L2
// at N = 2048, q = 64).
template <int Q, int MODE, int WAVES, int EX, bool REC>
__global__ __launch_bounds__(64 * WAVES) void k_fwd(SweepArgs a) {
  using C = Cfg<Q, WAVES>;
  using Lt = Lay<Q, EX>;
  using V = typename Lt::V;
  constexpr int NB = Lt::NB, NV = Lt::NV;
  __shared__ float W[2][C::WSZ];
  __shared__ double red[WAVES];
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.y;
  const int Nc = gridDim.y;
  const int e = (blockIdx.x * WAVES + (threadIdx.x >> 6)) * EX + (lane % EX);
  const bool on = e < a.B;
  const size_t slice = (size_t)a.B * Q;
  const size_t row = (size_t)(on ? e : 0) * Q + 4 * (lane / EX);
  const float* K = static_cast<const float*>(a.K);
  const float* bb = static_cast<const float*>(a.b);
  float* X = static_cast<float*>(a.X);
  const float* G = static_cast<const float*>(a.G);
  const float* Cs = static_cast<const float*>(a.Cs);
  const float* Vn = static_cast<const float*>(a.V);
  const int c = a.c;
  const int nsteps = MODE == SWEEP_CORRF ? c - 1 : c;
  const float hl = (float)a.hl, hc = (float)a.hc;
  const long kc = (long)k * c;

  WRegs<Q, WAVES> wr;
  w_fetch<Q, WAVES>(wr, K, bb, (size_t)kc * a.stride);
  w_put<Q, WAVES>(W[0], wr);
  __syncthreads();

  V v[NB];
#pragma unroll
  for (int mb = 0; mb < NB; ++mb) v[mb] = 0.f;
  if (on) {
    if (MODE == SWEEP_FC) {
      // a pending coarse-grid correction of the previous cycle is applied on the fly
      if (MODE == SWEEP_FC && Vn)
        correct<Lt>(v, Cs + (size_t)k * a.cs_stride * slice + row, Vn + (size_t)k * slice + row);
      else Lt::load(v, X + kc * slice + row);
      if (MODE == SWEEP_FC && k == 0) Lt::store(static_cast<float*>(a.S) + row, v);
    } else if (MODE == SWEEP_FRES) {
      Lt::load(v, Cs + (size_t)k * a.cs_stride * slice + row);
    } else {
      correct<Lt>(v, Cs + (size_t)k * a.cs_stride * slice + row, Vn + (size_t)k * slice + row);
      if (k > 0) Lt::store(X + kc * slice + row, v);
    }
  }
  V coarse[NB];
  // the final F-relaxation records sigma'(z) of every layer, and also takes the
  // product of the layer before the next C-point
  constexpr bool rec = REC && MODE == SWEEP_CORRF;
  constexpr int extra = rec ? 1 : 0;
  for (int j = 0; j < nsteps; ++j) {
    // prefetch the next layer (the last step re-fetches its own, or the extra one)
    w_fetch<Q, WAVES>(wr, K, bb, (size_t)(kc + (j + 1 < nsteps ? j + 1 : j + extra)) * a.stride);
    V s[NB];
    Lt::template prod<C::LD>(s, v, W[j & 1], lane);
    if constexpr (rec) {
      V dz[NB];
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) dz[mb] = s[mb];
      apply<V, NB, NV>(dz, a.act, true);
      store_dsig<Lt>(a.dsig, (size_t)(kc + j) * a.stride * slice + row, a.act, dz, on);
    }
    apply<V, NB, NV>(s, a.act, false);
    if (MODE == SWEEP_FRES && j == 0) {
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) coarse[mb] = v[mb] + hc * s[mb];
    }
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) v[mb] = v[mb] + hl * s[mb];
    if (on) {
      if (G) {
        V t[NB];
        Lt::load(t, G + (kc + j + 1) * slice + row);
        add_to<V, NB>(v, t);
      }
      if (MODE == SWEEP_CORRF) Lt::store(X + (kc + j + 1) * slice + row, v);
    }
    w_put<Q, WAVES>(W[(j + 1) & 1], wr);
    __syncthreads();
  }

  if constexpr (extra != 0) {
    // sigma' of the layer before the next C-point, from the last F-point
    V z[NB];
    Lt::template prod<C::LD>(z, v, W[nsteps & 1], lane);
    apply<V, NB, NV>(z, a.act, true);
    store_dsig<Lt>(a.dsig, (size_t)(kc + nsteps) * a.stride * slice + row, a.act, z, on);
  }
  if (MODE == SWEEP_FC) {
    if (on) Lt::store(static_cast<float*>(a.S) + (size_t)(k + 1) * slice + row, v);
  } else if (MODE == SWEEP_FRES) {
    double acc = 0.0;
    if (on) {
      V cn[NB];
      Lt::load(cn, Cs + (size_t)(k + 1) * a.cs_stride * slice + row);
      acc = sq_diff<V, NB, NV>(v, cn);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) coarse[mb] = v[mb] - coarse[mb];  // g_{l+1}^{k+1}
      Lt::store(static_cast<float*>(a.Gn) + (size_t)(k + 1) * slice + row, coarse);
      if (a.xn_every > 0 && (k + 1) % a.xn_every == 0)
        Lt::store(static_cast<float*>(a.Xn) + (size_t)(k + 1) * slice + row, cn);
      if (k == 0) {
        Lt::load(cn, Cs + row);
        Lt::store(static_cast<float*>(a.Xn) + row, cn);
      }
    }
    if (a.partial) {
      const double s = wg_sum<WAVES>(acc, red);
      if (threadIdx.x == 0) a.partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
    }
  } else if (MODE == SWEEP_CORRF) {
    if (on && k == Nc - 1) {
      correct<Lt>(v, Cs + (size_t)Nc * a.cs_stride * slice + row, Vn + (size_t)Nc * slice + row);
      Lt::store(X + (size_t)a.Nl * slice + row, v);
    }
  }
}

// ------------------------------------------------------------------ adjoint
// Interval k runs from its upper C-point (k+1)c down to kc; step j produces level
// point i = (k+1)c-1-j, linearised at the fine state of index i*stride.
template <int Q, int MODE, int WAVES, int EX, bool REC>
__global__ __launch_bounds__(64 * WAVES)
__attribute__((amdgpu_waves_per_eu(Q == 64 && REC ? (MODE == SWEEP_FRES ? 3 : 4) : 1, 8))) void k_adj(SweepArgs a) {
  using C = Cfg<Q, WAVES>;
  using Lt = Lay<Q, EX>;
  using V = typename Lt::V;
  constexpr int NB = Lt::NB, NV = Lt::NV;
  __shared__ float W[2][C::WSZ];
  __shared__ double red[WAVES];
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.y;
  const int Nc = gridDim.y;
  const int e = (blockIdx.x * WAVES + (threadIdx.x >> 6)) * EX + (lane % EX);
  const bool on = e < a.B;
  const size_t slice = (size_t)a.B * Q;
  const size_t row = (size_t)(on ? e : 0) * Q + 4 * (lane / EX);
  const float* K = static_cast<const float*>(a.K);
  const float* bb = static_cast<const float*>(a.b);
  const float* Uf = static_cast<const float*>(a.Uf);
  float* X = static_cast<float*>(a.X);
  const float* G = static_cast<const float*>(a.G);
  const float* Cs = static_cast<const float*>(a.Cs);
  const float* Vn = static_cast<const float*>(a.V);
  const int c = a.c;
  const int nsteps = MODE == SWEEP_CORRF ? c - 1 : c;
  const float hl = (float)a.hl, hc = (float)a.hc;
  const long top = (long)(k + 1) * c;

  WRegs<Q, WAVES> wr;
  w_fetch<Q, WAVES>(wr, K, bb, (size_t)(top - 1) * a.stride);
  w_put<Q, WAVES>(W[0], wr);
  __syncthreads();

  V v[NB], cu[NB];
#pragma unroll
  for (int mb = 0; mb < NB; ++mb) v[mb] = 0.f;
  if (on) {
    if (MODE == SWEEP_FC) {
      if (Vn)
        correct<Lt>(v, Cs + (size_t)(k + 1) * a.cs_stride * slice + row, Vn + (size_t)(k + 1) * slice + row);
      else Lt::load(v, X + top * slice + row);
      if (MODE == SWEEP_FC && k == Nc - 1) Lt::store(static_cast<float*>(a.S) + (size_t)Nc * slice + row, v);
    } else if (MODE == SWEEP_FRES) {
      Lt::load(v, Cs + (size_t)(k + 1) * a.cs_stride * slice + row);
    } else {
      correct<Lt>(v, Cs + (size_t)(k + 1) * a.cs_stride * slice + row, Vn + (size_t)(k + 1) * slice + row);
      if (k + 1 < Nc) Lt::store(X + top * slice + row, v);
    }
  }
  if (MODE == SWEEP_FRES) {
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) cu[mb] = v[mb];
  }
  constexpr bool rec = REC;  // sigma' from the record instead of K u + b
  // at width 64 the record row of the next step is requested one step ahead
  // (the extra registers do not lower the occupancy there)
  constexpr bool PFR = rec && Q == 64;
  V rn[NB];
  if (PFR) load_dsig<Lt>(rn, a.dsig, (size_t)(top - 1) * a.stride * slice + row, a.act);
  for (int j = 0; j < nsteps; ++j) {
    const long i = top - 1 - j;
    w_fetch<Q, WAVES>(wr, K, bb, (size_t)(j + 1 < nsteps ? i - 1 : i) * a.stride);
    V d[NB], w[NB];
    if constexpr (rec) {
      // every lane reads a valid row; columns of lanes past the batch are never stored
      if constexpr (PFR) {
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) d[mb] = rn[mb];
        if (j + 1 < nsteps) load_dsig<Lt>(rn, a.dsig, (size_t)(i - 1) * a.stride * slice + row, a.act);
      } else {
        load_dsig<Lt>(d, a.dsig, (size_t)i * a.stride * slice + row, a.act);
      }
    } else {
      V u[NB];
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) u[mb] = 0.f;
      if (on) Lt::load(u, Uf + (size_t)i * a.ustride * slice + row);
      Lt::template prod<C::LD>(d, u, W[j & 1], lane);
      apply<V, NB, NV>(d, a.act, true);
    }
    if (MODE == SWEEP_FRES && j == nsteps - 1) {
      // coarse adjoint step from the upper C-point, linearised at the same fine state
      V s2[NB];
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) s2[mb] = d[mb] * cu[mb];
      Lt::template prod_t<C::LD>(w, s2, W[j & 1], lane);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) cu[mb] = cu[mb] + hc * w[mb];
    }
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) d[mb] = d[mb] * v[mb];
    Lt::template prod_t<C::LD>(w, d, W[j & 1], lane);
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) v[mb] = v[mb] + hl * w[mb];
    if (on) {
      if (G) {
        V t[NB];
        Lt::load(t, G + (size_t)i * slice + row);
        add_to<V, NB>(v, t);
      }
      if (MODE == SWEEP_CORRF) Lt::store(X + (size_t)i * slice + row, v);
    }
    w_put<Q, WAVES>(W[(j + 1) & 1], wr);
    __syncthreads();
  }

  if (MODE == SWEEP_FC) {
    if (on) Lt::store(static_cast<float*>(a.S) + (size_t)k * slice + row, v);
  } else if (MODE == SWEEP_FRES) {
    double acc = 0.0;
    if (on) {
      V ck[NB];
      Lt::load(ck, Cs + (size_t)k * a.cs_stride * slice + row);
      acc = sq_diff<V, NB, NV>(v, ck);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) cu[mb] = v[mb] - cu[mb];  // g_{l+1}^k
      Lt::store(static_cast<float*>(a.Gn) + (size_t)k * slice + row, cu);
      if (a.xn_every > 0 && k % a.xn_every == 0)
        Lt::store(static_cast<float*>(a.Xn) + (size_t)k * slice + row, ck);
      if (k == Nc - 1) {
        Lt::load(ck, Cs + (size_t)Nc * a.cs_stride * slice + row);
        Lt::store(static_cast<float*>(a.Xn) + (size_t)Nc * slice + row, ck);
      }
    }
    if (a.partial) {
      const double s = wg_sum<WAVES>(acc, red);
      if (threadIdx.x == 0) a.partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
    }
  } else if (MODE == SWEEP_CORRF) {
    if (on && k == 0) {
      correct<Lt>(v, Cs + row, Vn + row);
      Lt::store(X + row, v);
    }
  }
}

// ------------------------------------------------------------------ interval-resident sweeps
// With c = 4 the sweeps of the width-32 layers are latency-bound when every step
// waits on its own rows behind a barrier. These variants stage the weights of all
// the interval's layers in LDS at once and request every row the interval reads
// (right-hand-side rows, sigma' record or primal rows, the second C-point) before
// the first step, so a workgroup waits on memory about once, and the step loop
// has no barrier. Arithmetic and operand order are those of k_fwd / k_adj, step
// by step. Lanes past the batch read example 0's rows (valid memory) and store
// nothing; in the matrix-core products every example is its own column, so those
// lanes do not touch the others' results.
constexpr int IV_CF = 4;

// Weights and biases of NL consecutive layers in flight between global memory and LDS.
template <int Q, int NL, int WAVES>
struct WAll {
  static constexpr int NT = 64 * WAVES;
  static constexpr int KV = Q * Q / 4;  // float4 slots of one K_n
  static constexpr int BV = Q / 4;      // float4 slots of one b_n
  static constexpr int PK = (NL * KV + NT - 1) / NT;
  static constexpr int PB = (NL * BV + NT - 1) / NT;
  f32x4 k[PK];
  f32x4 b[PB];
};

// Slot j holds fine layer (n0 + dn j) * stride.
template <int Q, int NL, int WAVES>
__device__ __forceinline__ void wall_fetch(WAll<Q, NL, WAVES>& r, const float* __restrict__ K,
                                           const float* __restrict__ b, long n0, long dn, long stride) {
  using A = WAll<Q, NL, WAVES>;
#pragma unroll
  for (int p = 0; p < A::PK; ++p) {
    const int idx = threadIdx.x + p * A::NT;
    if (idx < NL * A::KV) {
      const int j = idx / A::KV, w = idx - j * A::KV;
      r.k[p] = reinterpret_cast<const f32x4g*>(K + (size_t)((n0 + dn * j) * stride) * (Q * Q))[w];
    }
  }
#pragma unroll
  for (int p = 0; p < A::PB; ++p) {
    const int idx = threadIdx.x + p * A::NT;
    if (idx < NL * A::BV) {
      const int j = idx / A::BV, w = idx - j * A::BV;
      r.b[p] = reinterpret_cast<const f32x4g*>(b + (size_t)((n0 + dn * j) * stride) * Q)[w];
    }
  }
}

template <int Q, int NL, int WAVES>
__device__ __forceinline__ void wall_put(float* sh, const WAll<Q, NL, WAVES>& r) {
  using A = WAll<Q, NL, WAVES>;
  using C = Cfg<Q, WAVES>;
#pragma unroll
  for (int p = 0; p < A::PK; ++p) {
    const int idx = threadIdx.x + p * A::NT;
    if (idx < NL * A::KV) {
      const int j = idx / A::KV, w = idx - j * A::KV;
      const int el = w * 4, row = el / Q, col = el - row * Q;
      *reinterpret_cast<f32x4*>(sh + j * C::WSZ + row * C::LD + col) = r.k[p];
    }
  }
#pragma unroll
  for (int p = 0; p < A::PB; ++p) {
    const int idx = threadIdx.x + p * A::NT;
    if (idx < NL * A::BV) {
      const int j = idx / A::BV, w = idx - j * A::BV;
      *reinterpret_cast<f32x4*>(sh + j * C::WSZ + Q * C::LD + w * 4) = r.b[p];
    }
  }
}

// The interval kernels can walk batch tiles: workgroup (g, k) stages the weights
// of interval k once and runs tiles g, g + gridDim.x, ... of 64 examples (tile
// mode TM = 1), so the weights are read from L2 once per workgroup instead of once
// per tile; with TM = 2 the rows of its next tile are requested before the current
// tile's steps (the index is clamped, so every load is issued unconditionally and
// the waits stay exact) and a tile's loads overlap the previous tile's products.
// TM = 0 is one tile per workgroup.
__device__ __forceinline__ size_t iv_row(int t, int waves, int ex, int B, int Q, bool& on) {
  const int lane = threadIdx.x & 63;
  const int e = (t * waves + (threadIdx.x >> 6)) * ex + (lane % ex);
  on = e < B;
  return (size_t)(on ? e : 0) * Q + 4 * (lane / ex);
}

// Rows of one tile for a forward interval sweep: two state rows (FC: the C-point,
// or the staged C-point and the coarse value of a pending correction; FRES: the
// lower and the upper C-point; CORRF: the C-point and its coarse value) and the
// level's right-hand-side rows.
template <typename Lt, int NS, bool HASG>
struct FwdRows {
  typename Lt::V a[Lt::NB], c[Lt::NB];
  typename Lt::V g[HASG ? NS : 1][Lt::NB];
};

// REC: the final F-relaxation writes the sigma' record (CORRF only).
// HASG: the level has right-hand-side rows (every level but the finest).
template <int Q, int MODE, int WAVES, bool REC, bool HASG, int TM, bool CORR>
__global__ __launch_bounds__(64 * WAVES) void k_fwd_iv(SweepArgs a) {
  constexpr int EX = 16;
  using C = Cfg<Q, WAVES>;
  using Lt = Lay<Q, EX>;
  using V = typename Lt::V;
  constexpr int NB = Lt::NB, NV = Lt::NV;
  constexpr bool rec = REC && MODE == SWEEP_CORRF;
  constexpr int NS = MODE == SWEEP_CORRF ? IV_CF - 1 : IV_CF;
  constexpr int NL = NS + (rec ? 1 : 0);
  using Rows = FwdRows<Lt, NS, HASG>;
  __shared__ float W[NL * C::WSZ];
  __shared__ double red[WAVES];
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.y;
  const int Nc = gridDim.y;
  const int ntiles = (a.B + EX * WAVES - 1) / (EX * WAVES);
  const size_t slice = (size_t)a.B * Q;
  float* X = static_cast<float*>(a.X);
  const float* G = static_cast<const float*>(a.G);
  const float* Cs = static_cast<const float*>(a.Cs);
  const float* Vn = static_cast<const float*>(a.V);
  const float hl = (float)a.hl, hc = (float)a.hc;
  const long kc = (long)k * IV_CF;

  if (MODE == SWEEP_CORRF && !HASG && a.cpt) {
    // C-point storage: the corrected C-points are the whole result (the F-points
    // are not stored; the adjoint and the gradient recompute them from these)
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
      bool on;
      const size_t row = iv_row(t, WAVES, EX, a.B, Q, on);
      if (on) {
        V v[NB];
        if (k > 0) {
          correct<Lt>(v, Cs + (size_t)k * a.cs_stride * slice + row, Vn + (size_t)k * slice + row);
          Lt::store(X + (size_t)k * slice + row, v);
        }
        if (k == Nc - 1) {
          correct<Lt>(v, Cs + (size_t)Nc * a.cs_stride * slice + row, Vn + (size_t)Nc * slice + row);
          Lt::store(X + (size_t)Nc * slice + row, v);
        }
      }
    }
    return;
  }

  // FC with CORR (a.V set) reads its C-points as C + (V - C): a pending coarse-grid
  // correction of the previous cycle applied on the fly, or (the second FC sweep of
  // FCFCF) staged C-points read as C + (C - C); with C-point storage C-point k is
  // row k of the level-0 trajectory
  constexpr bool pair = MODE != SWEEP_FC || CORR;
  auto load_rows = [&](Rows& r, size_t row) {
    if (MODE == SWEEP_FC && !pair) {
      Lt::load(r.a, X + (a.cpt ? (long)k : kc) * slice + row);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) r.c[mb] = 0.f;  // unused; initialised so the rows stay in registers
    } else {
      Lt::load(r.a, Cs + (size_t)k * a.cs_stride * slice + row);
      if (MODE == SWEEP_FRES) Lt::load(r.c, Cs + (size_t)(k + 1) * a.cs_stride * slice + row);
      else Lt::load(r.c, Vn + (size_t)k * slice + row);
    }
    if constexpr (HASG) {
#pragma unroll
      for (int j = 0; j < NS; ++j) Lt::load(r.g[j], G + (kc + j + 1) * slice + row);
    }
  };

  WAll<Q, NL, WAVES> wr;
  wall_fetch<Q, NL, WAVES>(wr, static_cast<const float*>(a.K), static_cast<const float*>(a.b), kc, 1, a.stride);
  Rows cur;
  {
    bool on0;
    load_rows(cur, iv_row(blockIdx.x, WAVES, EX, a.B, Q, on0));
  }
  wall_put<Q, NL, WAVES>(W, wr);
  __syncthreads();

  double acc = 0.0;
  // the work of one tile t, reading the staged weights through Wt
  auto tile = [&](Rows& cur, int t, const float* Wt) {
    bool on;
    const size_t row = iv_row(t, WAVES, EX, a.B, Q, on);
    V v[NB];
    if (MODE == SWEEP_FC && !pair) {
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = cur.a[mb];
    } else if (MODE == SWEEP_FRES) {
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = cur.a[mb];
    } else {
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = cur.a[mb] + (cur.c[mb] - cur.a[mb]);  // C + (V - C)
    }
    if (on) {
      if (MODE == SWEEP_FC && k == 0) Lt::store(static_cast<float*>(a.S) + row, v);
      if (MODE == SWEEP_CORRF && k > 0) Lt::store(X + kc * slice + row, v);
    }

    V coarse[NB];
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      V s[NB];
      Lt::template prod<C::LD>(s, v, Wt + j * C::WSZ, lane);
      if constexpr (rec) {
        V dz[NB];
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) dz[mb] = s[mb];
        apply<V, NB, NV>(dz, a.act, true);
        store_dsig<Lt>(a.dsig, (size_t)(kc + j) * a.stride * slice + row, a.act, dz, on);
      }
      apply<V, NB, NV>(s, a.act, false);
      if (MODE == SWEEP_FRES && j == 0) {
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) coarse[mb] = v[mb] + hc * s[mb];
      }
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = v[mb] + hl * s[mb];
      if constexpr (HASG) add_to<V, NB>(v, cur.g[j]);
      if (MODE == SWEEP_CORRF && on) Lt::store(X + (kc + j + 1) * slice + row, v);
    }

    if constexpr (rec) {
      // sigma' of the layer before the next C-point, from the last F-point
      V z[NB];
      Lt::template prod<C::LD>(z, v, Wt + NS * C::WSZ, lane);
      apply<V, NB, NV>(z, a.act, true);
      store_dsig<Lt>(a.dsig, (size_t)(kc + NS) * a.stride * slice + row, a.act, z, on);
    }
    if (MODE == SWEEP_FC) {
      if (on) Lt::store(static_cast<float*>(a.S) + (size_t)(k + 1) * slice + row, v);
    } else if (MODE == SWEEP_FRES) {
      if (on) {
        acc += sq_diff<V, NB, NV>(v, cur.c);
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) coarse[mb] = v[mb] - coarse[mb];  // g_{l+1}^{k+1}
        Lt::store(static_cast<float*>(a.Gn) + (size_t)(k + 1) * slice + row, coarse);
        if (a.xn_every > 0 && (k + 1) % a.xn_every == 0)
          Lt::store(static_cast<float*>(a.Xn) + (size_t)(k + 1) * slice + row, cur.c);
        if (k == 0) {
          V c0[NB];
          Lt::load(c0, Cs + row);
          Lt::store(static_cast<float*>(a.Xn) + row, c0);
        }
      }
    } else if (MODE == SWEEP_CORRF) {
      if (on && k == Nc - 1) {
        correct<Lt>(v, Cs + (size_t)Nc * a.cs_stride * slice + row, Vn + (size_t)Nc * slice + row);
        Lt::store(X + (size_t)a.Nl * slice + row, v);
      }
    }
  };
  if constexpr (TM == 0) {
    tile(cur, blockIdx.x, W);
  } else {
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
      // the products read the staged weights from LDS in every tile: an offset
      // the compiler cannot see through keeps it from hoisting those reads out of
      // the loop into registers
      int woff = 0;
      asm volatile("" : "+v"(woff));
      Rows nxt;
      if constexpr (TM == 2) {
        bool on1;
        load_rows(nxt, iv_row(min(t + (int)gridDim.x, ntiles - 1), WAVES, EX, a.B, Q, on1));
      } else if (t != (int)blockIdx.x) {
        bool on1;
        load_rows(cur, iv_row(t, WAVES, EX, a.B, Q, on1));
      }
      tile(cur, t, W + woff);
      if constexpr (TM == 2) cur = nxt;
    }
  }
  if (MODE == SWEEP_FRES && a.partial) {
    const double s = wg_sum<WAVES>(acc, red);
    if (threadIdx.x == 0) a.partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
  }
}

// Rows of one tile for an adjoint interval sweep: the two state rows (the upper
// C-point, or the staged C-point and coarse value of a correction; FRES: the upper
// and the lower C-point), what each step is linearised at (record rows, primal
// rows, or the lower primal C-point), and the right-hand-side rows.
template <typename Lt, int NS, bool REC, bool RBITS, bool CPT, bool HASG>
struct AdjRows {
  typename Lt::V a[Lt::NB], c[Lt::NB];
  RecRow<Lt, RBITS> rr[REC ? NS : 1];
  typename Lt::V u[(REC || CPT) ? 1 : NS][Lt::NB];
  typename Lt::V g[HASG ? NS : 1][Lt::NB];
};

// REC: sigma' comes from the record (ReLU: RBITS, one bit per value) instead of
// the layer product at the primal state.
// CPT (finest level, C-point storage): Uf holds the fine C-points only (row k is
// u^{kc}); the interval first recomputes its F-point states and sigma'(z_n) for
// n = kc .. kc + 3 by forward steps from its lower C-point, with the arithmetic of
// the forward F-relaxation (so the results equal those of full storage bit for bit).
// TM: tiles per workgroup (0: one; 1: several; 2: several, each one's rows
// requested during the previous one's steps). CORR: FC reads C + (V - C).
//
// Resident waves per SIMD the compiler must allow for. Width 32, finest level, bit
// record, one tile: eight. Width 64: two, which is what LDS allows (70 KB of weights
// per workgroup, two workgroups per CU); left to itself the compiler gives the
// fp32-record sweeps 260 registers, one wave per SIMD. The recomputing FRES sweeps
// that walk tiles are left free: held to 256 registers they spill.
template <int Q, int MODE, bool REC, bool RBITS, bool HASG, bool CPT, int TM>
constexpr int adj_iv_waves() {
  if (Q == 32) return !HASG && REC && RBITS && TM == 0 ? 8 : 1;
  if (Q == 64) return MODE == SWEEP_FRES && !REC && !CPT && TM != 0 ? 1 : 2;
  return 1;
}

template <int Q, int MODE, int WAVES, bool REC, bool RBITS, bool HASG, bool CPT, int TM, bool CORR>
__global__ __launch_bounds__(64 * WAVES)
__attribute__((amdgpu_waves_per_eu(adj_iv_waves<Q, MODE, REC, RBITS, HASG, CPT, TM>(), 8)))
void k_adj_iv(SweepArgs a) {
  static_assert(!(CPT && (REC || HASG)), "C-point storage is a finest-level mode without a record");
  constexpr int EX = 16;
  using C = Cfg<Q, WAVES>;
  using Lt = Lay<Q, EX>;
  using V = typename Lt::V;
  constexpr int NB = Lt::NB, NV = Lt::NV;
  constexpr int NS = MODE == SWEEP_CORRF ? IV_CF - 1 : IV_CF;
  constexpr int NW = CPT ? IV_CF : NS;  // layers staged: the recompute needs all of the interval's
  // at eight waves per SIMD (width 32, finest level, bit record, no prefetch) the
  // registers go to occupancy, and FRES reads its lower C-point after the steps
  constexpr bool LATE_CK = MODE == SWEEP_FRES && Q == 32 && !HASG && REC && RBITS && TM == 0;
  using Rows = AdjRows<Lt, NS, REC, RBITS, CPT, HASG>;
  __shared__ float W[NW * C::WSZ];
  __shared__ double red[WAVES];
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.y;
  const int Nc = gridDim.y;
  const int ntiles = (a.B + EX * WAVES - 1) / (EX * WAVES);
  const size_t slice = (size_t)a.B * Q;
  const float* Uf = static_cast<const float*>(a.Uf);
  float* X = static_cast<float*>(a.X);
  const float* G = static_cast<const float*>(a.G);
  const float* Cs = static_cast<const float*>(a.Cs);
  const float* Vn = static_cast<const float*>(a.V);
  const float hl = (float)a.hl, hc = (float)a.hc;
  const long top = (long)(k + 1) * IV_CF;

  // step j is linearised at fine index (top - 1 - j) * stride, the primal state of
  // which is row (top - 1 - j) * ustride of Uf
  constexpr bool pair = MODE != SWEEP_FC || CORR;  // FC reading C + (V - C), as in k_fwd_iv
  auto load_rows = [&](Rows& r, size_t row) {
    if (MODE == SWEEP_FC && !pair) {
      Lt::load(r.a, X + top * slice + row);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) r.c[mb] = 0.f;  // unused; initialised so the rows stay in registers
    } else {
      Lt::load(r.a, Cs + (size_t)(k + 1) * a.cs_stride * slice + row);
      if (MODE == SWEEP_FRES) {
        if (!LATE_CK) Lt::load(r.c, Cs + (size_t)k * a.cs_stride * slice + row);
      } else {
        Lt::load(r.c, Vn + (size_t)(k + 1) * slice + row);
      }
    }
    if constexpr (REC) {
#pragma unroll
      for (int j = 0; j < NS; ++j) r.rr[j].load(a.dsig, (size_t)(top - 1 - j) * a.stride * slice + row);
    } else if constexpr (CPT) {
      Lt::load(r.u[0], Uf + (size_t)k * slice + row);  // u^{kc}
    } else {
#pragma unroll
      for (int j = 0; j < NS; ++j) Lt::load(r.u[j], Uf + (size_t)(top - 1 - j) * a.ustride * slice + row);
    }
    if constexpr (HASG) {
#pragma unroll
      for (int j = 0; j < NS; ++j) Lt::load(r.g[j], G + (size_t)(top - 1 - j) * slice + row);
    }
  };

  WAll<Q, NW, WAVES> wr;  // slot j holds layer top - 1 - j
  wall_fetch<Q, NW, WAVES>(wr, static_cast<const float*>(a.K), static_cast<const float*>(a.b), top - 1, -1,
                           a.stride);
  Rows cur;
  {
    bool on0;
    load_rows(cur, iv_row(blockIdx.x, WAVES, EX, a.B, Q, on0));
  }
  wall_put<Q, NW, WAVES>(W, wr);
  __syncthreads();

  double acc = 0.0;
  // the work of one tile t, reading the staged weights through Wt
  auto tile = [&](Rows& cur, int t, const float* Wt) {
    bool on;
    const size_t row = iv_row(t, WAVES, EX, a.B, Q, on);
    // C-point storage: dz[jf] = sigma'(z_{kc+jf}) along u^{kc+jf+1} = u^{kc+jf} + h sigma(z_{kc+jf})
    V dz[CPT ? IV_CF : 1][NB];
    if constexpr (CPT) {
#pragma unroll
      for (int jf = 0; jf < IV_CF; ++jf) {
        V sz[NB];
        Lt::template prod<C::LD, !HASG>(sz, cur.u[0], Wt + (IV_CF - 1 - jf) * C::WSZ, lane);
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) dz[jf][mb] = sz[mb];
        apply<V, NB, NV>(dz[jf], a.act, true);
        if (jf + 1 < IV_CF) {
          apply<V, NB, NV>(sz, a.act, false);
#pragma unroll
          for (int mb = 0; mb < NB; ++mb) cur.u[0][mb] = cur.u[0][mb] + hl * sz[mb];
        }
      }
    }
    V v[NB], cu[NB];
    if (MODE == SWEEP_FC && !pair) {
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = cur.a[mb];
    } else if (MODE == SWEEP_FRES) {
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = cu[mb] = cur.a[mb];
    } else {
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = cur.a[mb] + (cur.c[mb] - cur.a[mb]);  // C + (V - C)
    }
    if (on) {
      if (MODE == SWEEP_FC && k == Nc - 1) Lt::store(static_cast<float*>(a.S) + (size_t)Nc * slice + row, v);
      if (MODE == SWEEP_CORRF && k + 1 < Nc) Lt::store(X + top * slice + row, v);
    }

#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const float* Wj = Wt + j * C::WSZ;
      V d[NB], w[NB];
      if constexpr (REC) {
        cur.rr[j].get(d);
      } else if constexpr (CPT) {
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) d[mb] = dz[IV_CF - 1 - j][mb];
      } else {
        Lt::template prod<C::LD, !HASG>(d, cur.u[j], Wj, lane);
        apply<V, NB, NV>(d, a.act, true);
      }
      if (MODE == SWEEP_FRES && j == NS - 1) {
        // coarse adjoint step from the upper C-point, linearised at the same fine state
        V s2[NB];
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) s2[mb] = d[mb] * cu[mb];
        Lt::template prod_t<C::LD, !HASG>(w, s2, Wj, lane);
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) cu[mb] = cu[mb] + hc * w[mb];
      }
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) d[mb] = d[mb] * v[mb];
      Lt::template prod_t<C::LD, !HASG>(w, d, Wj, lane);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = v[mb] + hl * w[mb];
      if constexpr (HASG) add_to<V, NB>(v, cur.g[j]);
      if (MODE == SWEEP_CORRF && on) Lt::store(X + (size_t)(top - 1 - j) * slice + row, v);
    }

    if (MODE == SWEEP_FC) {
      if (on) Lt::store(static_cast<float*>(a.S) + (size_t)k * slice + row, v);
    } else if (MODE == SWEEP_FRES) {
      if (on) {
        if (LATE_CK) Lt::load(cur.c, Cs + (size_t)k * a.cs_stride * slice + row);
        acc += sq_diff<V, NB, NV>(v, cur.c);
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) cu[mb] = v[mb] - cu[mb];  // g_{l+1}^k
        Lt::store(static_cast<float*>(a.Gn) + (size_t)k * slice + row, cu);
        if (a.xn_every > 0 && k % a.xn_every == 0)
          Lt::store(static_cast<float*>(a.Xn) + (size_t)k * slice + row, cur.c);
        if (k == Nc - 1) {
          V cN[NB];
          Lt::load(cN, Cs + (size_t)Nc * a.cs_stride * slice + row);
          Lt::store(static_cast<float*>(a.Xn) + (size_t)Nc * slice + row, cN);
        }
      }
    } else if (MODE == SWEEP_CORRF) {
      if (on && k == 0) {
        correct<Lt>(v, Cs + row, Vn + row);
        Lt::store(X + row, v);
      }
    }
  };
  if constexpr (TM == 0) {
    tile(cur, blockIdx.x, W);
  } else {
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
      // the products read the staged weights from LDS in every tile: an offset
      // the compiler cannot see through keeps it from hoisting those reads out of
      // the loop into registers
      int woff = 0;
      asm volatile("" : "+v"(woff));
      Rows nxt;
      if constexpr (TM == 2) {
        bool on1;
        load_rows(nxt, iv_row(min(t + (int)gridDim.x, ntiles - 1), WAVES, EX, a.B, Q, on1));
      } else if (t != (int)blockIdx.x) {
        bool on1;
        load_rows(cur, iv_row(t, WAVES, EX, a.B, Q, on1));
      }
      tile(cur, t, W + woff);
      if constexpr (TM == 2) cur = nxt;
    }
  }
  if (MODE == SWEEP_FRES && a.partial) {
    const double s = wg_sum<WAVES>(acc, red);
    if (threadIdx.x == 0) a.partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
  }
}

// ------------------------------------------------------------------ gradient
// Workgroup (layer n, batch chunk). Each wave takes 32 examples at a time:
// s = sigma'(K_n u + b_n) * lam^{n+1} in accumulator layout (one matrix-core
// product), then s and u go through LDS as [example][feature] tiles so that
// dK[i][j] += sum_e s[e][i] u[e][j] runs as a second product with the examples
// as the contraction index (k-slice t pairs examples 2t and 2t+1). db sums the s
// tile's columns. The four waves' accumulators are combined in a fixed order and
// written as the chunk's partial; a second pass sums the chunks in order and
// scales by h (deterministic).
constexpr int GRAD_WAVES = 4;

// With the record (REC) the layer weights are not needed (no forward product), so
// they are not staged: at width 64 the workgroup then takes 67 KB of LDS, two fit
// on a CU, and the kernel is held to two waves per SIMD (left free it takes about
// 276 registers, one wave, and each chunk's loads are waited on in full).
// Lanes of one wave exchanging data through LDS: a wave's LDS instructions run in
// order, so a compiler fence and a wave barrier are enough between the writes and
// the reads.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int Q, bool REC>
__global__ __launch_bounds__(64 * GRAD_WAVES) __attribute__((amdgpu_waves_per_eu(REC && Q == 64 ? 2 : 1, 8)))
void k_grad(GradArgs a) {
  using C = Cfg<Q, GRAD_WAVES>;
  constexpr int MB = C::MB;
  constexpr int TL = Q + 1;  // tile row (floats)
  __shared__ float W[REC ? 1 : C::WSZ];
  __shared__ float tile[GRAD_WAVES][2][32 * TL];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = lane >> 5, li = lane & 31;
  const long n = a.n0 + blockIdx.x;  // layer; its state is row blockIdx.x of U
  const int chunk = blockIdx.y;
  const int per = (((a.B + a.nchunks - 1) / a.nchunks) + 32 * GRAD_WAVES - 1) / (32 * GRAD_WAVES) *
                  (32 * GRAD_WAVES);
  const int e0 = chunk * per, e1 = min(a.B, e0 + per);
  const size_t slice = (size_t)a.B * Q;
  const float* U = static_cast<const float*>(a.U) + (size_t)blockIdx.x * slice;
  const float* L = static_cast<const float*>(a.Lam) + (size_t)(n + 1) * slice;
  if constexpr (!REC) {
    WRegs<Q, GRAD_WAVES> wr;
    w_fetch<Q, GRAD_WAVES>(wr, static_cast<const float*>(a.K), static_cast<const float*>(a.b), n);
    w_put<Q, GRAD_WAVES>(W, wr);
    __syncthreads();
  }
  f32x16 acc[MB][MB];
#pragma unroll
  for (int x = 0; x < MB; ++x)
#pragma unroll
    for (int y = 0; y < MB; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
  float dbacc = 0.f;  // lane < Q: column sum of s over this wave's examples
  float* st = tile[wave][0];
  float* ut = tile[wave][1];
  using Lt = Lay<Q, 32>;
  // the rows of the wave's 32 examples from base on (zero past the chunk)
  auto ld_rows = [&](int base, f32x16 (&u)[MB], f32x16 (&s)[MB]) {
    const int e = base + wave * 32 + li;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) u[mb] = s[mb] = 0.f;
    if (e < e1) {
      Lt::load(u, U + (size_t)e * Q + 4 * h);
      Lt::load(s, L + (size_t)e * Q + 4 * h);
    }
  };
  // At width 32 the next examples' rows are requested during the contraction
  // (their registers cost no occupancy there); the tiles are the wave's own, so
  // its lanes meet at wave barriers only.
  constexpr bool PF = Q == 32;
  f32x16 un[PF ? MB : 1], sn[PF ? MB : 1];
  if constexpr (PF) ld_rows(e0, un, sn);
  for (int base = e0; base < e1; base += 32 * GRAD_WAVES) {
    const int e = base + wave * 32 + li;
    const size_t row = (size_t)(e < e1 ? e : 0) * Q + 4 * h;
    f32x16 u[MB], s[MB];
    if constexpr (PF) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        u[mb] = un[mb];
        s[mb] = sn[mb];
      }
    } else {
      ld_rows(base, u, s);
    }
    {
      f32x16 z[MB];
      if constexpr (REC) {
        load_dsig<Lt>(z, a.dsig, (size_t)n * slice + row, a.act);
      } else {
        Lt::template prod<C::LD>(z, u, W, lane);
        apply<f32x16, MB, 16>(z, a.act, true);
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) s[mb] = z[mb] * s[mb];
    }
    // accumulator layout -> [example][feature] tiles
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int f = 32 * mb + 8 * (r >> 2) + 4 * h + (r & 3);
        st[li * TL + f] = s[mb][r];
        ut[li * TL + f] = u[mb][r];
      }
    if constexpr (PF) {
      wave_lds_sync();
      if (base + 32 * GRAD_WAVES < e1) ld_rows(base + 32 * GRAD_WAVES, un, sn);
    } else {
      __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int er = (2 * t + h) * TL + li;
#pragma unroll
      for (int x = 0; x < MB; ++x) {
        const float av = st[er + 32 * x];
#pragma unroll
        for (int y = 0; y < MB; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, ut[er + 32 * y], acc[x][y], 0, 0, 0);
      }
    }
    if (lane < Q)
      for (int t = 0; t < 32; ++t) dbacc += st[t * TL + lane];
    if constexpr (PF) wave_lds_sync();
    else __syncthreads();
  }
  if constexpr (PF) __syncthreads();  // the combine below reuses every wave's tiles
  // combine the waves in order: wave w adds its accumulators into a Q x Q buffer
  float* red = &tile[0][0][0];  // Q*Q + Q floats fit in the tiles
  for (int w = 0; w < GRAD_WAVES; ++w) {
    if (wave == w) {
#pragma unroll
      for (int x = 0; x < MB; ++x)
#pragma unroll
        for (int y = 0; y < MB; ++y)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int i = 32 * x + 8 * (r >> 2) + 4 * h + (r & 3), j = 32 * y + li;
            red[i * Q + j] = (w == 0 ? 0.f : red[i * Q + j]) + acc[x][y][r];
          }
      if (lane < Q) red[Q * Q + lane] = (w == 0 ? 0.f : red[Q * Q + lane]) + dbacc;
    }
    __syncthreads();
  }
  float* out = static_cast<float*>(a.partial) + ((size_t)n * a.nchunks + chunk) * (Q * Q + Q);
  for (int o = threadIdx.x; o < Q * Q + Q; o += 64 * GRAD_WAVES) out[o] = red[o];
}

// Sum the chunk partials in chunk order in fp64 and scale by h.
__global__ __launch_bounds__(256) void k_grad_final(GradArgs a, int nw, int nbias) {
  const int nout = nw + nbias;
  const size_t o = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (o >= (size_t)a.N * nout) return;
  const size_t n = o / nout, r = o - n * nout;
  const float* p = static_cast<const float*>(a.partial) + n * a.nchunks * nout + r;
  double s = 0.0;
  for (int ch = 0; ch < a.nchunks; ++ch) s += (double)p[(size_t)ch * nout];
  const float v = (float)(s * a.h);
  if (r < (size_t)nw) static_cast<float*>(a.dK)[n * nw + r] = v;
  else static_cast<float*>(a.db)[n * nbias + (r - nw)] = v;
}

// First pass over `nl` layers starting at a.n0 (grid: layers x chunks).
template <int Q>
hipError_t grad_partials(const GradArgs& a, long nl, hipStream_t st) {
  // at width 32 the kernel is HBM-bound: an fp32 record row read per layer costs
  // more than the forward product it replaces, ReLU's bit record (1/32 of a row)
  // does not
  const bool rec = a.dsig && (Q >= 64 || a.act == ACT_RELU);
  if (rec) launch(k_grad<Q, true>, dim3((unsigned)nl, a.nchunks), 64 * GRAD_WAVES, 0, st, a);
  else launch(k_grad<Q, false>, dim3((unsigned)nl, a.nchunks), 64 * GRAD_WAVES, 0, st, a);
  return hipGetLastError();
}

template <int Q>
hipError_t grad_finish(const GradArgs& a, hipStream_t st) {
  const size_t tot = (size_t)a.N * (Q * Q + Q);
  launch(k_grad_final, (unsigned)((tot + 255) / 256), 256, 0, st, a, Q * Q, Q);
  return hipGetLastError();
}

template <int Q>
hipError_t grad(const GradArgs& a, hipStream_t st) {
  hipError_t err = grad_partials<Q>(a, a.N, st);
  if (err != hipSuccess) return err;
  return grad_finish<Q>(a, st);
}

// C-point storage: the F-relaxation of interval k0 + blockIdx.y from its lower
// C-point Uc[k0 + blockIdx.y], written to rows 4 blockIdx.y .. 4 blockIdx.y + 3 of Y
// (the C-point, then its three F-points), with the arithmetic of the forward
// sweeps' F-relaxation on the finest level (k_fwd_iv), so the states are those a
// full-storage solve stores.
template <int Q>
__global__ __launch_bounds__(64 * 4) void k_expand(const float* __restrict__ K, const float* __restrict__ bias,
                                                   const float* __restrict__ Uc, float* __restrict__ Y, int B,
                                                   long k0, float hl, int act) {
  constexpr int WAVES = 4, EX = 16, NL = IV_CF - 1;
  using C = Cfg<Q, WAVES>;
  using Lt = Lay<Q, EX>;
  using V = typename Lt::V;
  constexpr int NB = Lt::NB, NV = Lt::NV;
  __shared__ float W[NL * C::WSZ];
  const int lane = threadIdx.x & 63;
  const long k = k0 + blockIdx.y, kc = k * IV_CF;
  const int e = (blockIdx.x * WAVES + (threadIdx.x >> 6)) * EX + (lane % EX);
  const bool on = e < B;
  const size_t slice = (size_t)B * Q;
  const size_t row = (size_t)(on ? e : 0) * Q + 4 * (lane / EX);
  float* Yk = Y + (size_t)blockIdx.y * IV_CF * slice;
  WAll<Q, NL, WAVES> wr;
  wall_fetch<Q, NL, WAVES>(wr, K, bias, kc, 1, 1);
  V v[NB];
  Lt::load(v, Uc + (size_t)k * slice + row);
  wall_put<Q, NL, WAVES>(W, wr);
  __syncthreads();
  if (on) Lt::store(Yk + row, v);
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    V s[NB];
    Lt::template prod<C::LD>(s, v, W + j * C::WSZ, lane);
    apply<V, NB, NV>(s, act, false);
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) v[mb] = v[mb] + hl * s[mb];
    if (on) Lt::store(Yk + (size_t)(j + 1) * slice + row, v);
  }
}

constexpr int SWEEP_WAVES = 4;   // waves per interval workgroup (2 and 8 measured slower or equal)

// The sweeps run on the 16-example shape: measured faster than the 32-example
// one on every workload (q = 32 and 64, level 0 included), with fewer registers
// per wave and twice the waves.
constexpr int SWEEP_EX = 16;

// Interval-resident sweeps (c = 4): the level's right-hand side, the record kind
// and whether a workgroup prefetches its next tile select the instantiation.
template <int Q, bool HASG, int TM>
void sweep_iv(int dir, const SweepArgs& a, dim3 grid, hipStream_t st) {
  constexpr int W4 = SWEEP_WAVES;
  const bool rec = a.dsig != nullptr, bytes = a.act == ACT_RELU, corr = a.V != nullptr;
  if (dir == DIR_FWD) {
    if (a.mode == SWEEP_FC && corr) launch(k_fwd_iv<Q, SWEEP_FC, W4, false, HASG, TM, true>, grid, 64 * W4, 0, st, a);
    else if (a.mode == SWEEP_FC) launch(k_fwd_iv<Q, SWEEP_FC, W4, false, HASG, TM, false>, grid, 64 * W4, 0, st, a);
    else if (a.mode == SWEEP_FRES) launch(k_fwd_iv<Q, SWEEP_FRES, W4, false, HASG, TM, false>, grid, 64 * W4, 0, st, a);
    else if (rec) launch(k_fwd_iv<Q, SWEEP_CORRF, W4, true, HASG, TM, false>, grid, 64 * W4, 0, st, a);
    else launch(k_fwd_iv<Q, SWEEP_CORRF, W4, false, HASG, TM, false>, grid, 64 * W4, 0, st, a);
    return;
  }
#define LP_ADJ_IV(MODE, CORR)                                                                                         \
  do {                                                                                                                \
    if (!HASG && a.cpt) launch(k_adj_iv<Q, MODE, W4, false, false, false, true, TM, CORR>, grid, 64 * W4, 0, st, a);  \
    else if (!rec) launch(k_adj_iv<Q, MODE, W4, false, false, HASG, false, TM, CORR>, grid, 64 * W4, 0, st, a);       \
    else if (bytes) launch(k_adj_iv<Q, MODE, W4, true, true, HASG, false, TM, CORR>, grid, 64 * W4, 0, st, a);        \
    else launch(k_adj_iv<Q, MODE, W4, true, false, HASG, false, TM, CORR>, grid, 64 * W4, 0, st, a);                  \
  } while (0)
  if (a.mode == SWEEP_FC && corr) LP_ADJ_IV(SWEEP_FC, true);
  else if (a.mode == SWEEP_FC) LP_ADJ_IV(SWEEP_FC, false);
  else if (a.mode == SWEEP_FRES) LP_ADJ_IV(SWEEP_FRES, false);
  else LP_ADJ_IV(SWEEP_CORRF, false);
#undef LP_ADJ_IV
}

// LP_DENSE_SWEEP=staged keeps the double-buffered per-step kernels for c = 4 as
// well (for comparing the two designs).
bool iv_enabled() {
  static const bool on = [] {
    const char* e = getenv("LP_DENSE_SWEEP");
    return !(e && strcmp(e, "staged") == 0);
  }();
  return on;
}

// Which width-64 adjoint FRES sweeps run on the interval-resident kernel instead of
// the per-step one: LP_IV_FRES64 = 0 none, 1 the finest level's (the default:
// 51.1 against 55.7 ms per step on the deep workload; on coarse levels its record
// and right-hand-side rows leave one wave per SIMD), 2 every level's.
int iv_fres64() {
  static const int v = [] {
    const char* e = getenv("LP_IV_FRES64");
    return e ? atoi(e) : 1;
  }();
  return v;
}

// LP_IV_CORRF_WALK=1 lets the correction sweeps walk several tiles per workgroup
// as the other sweeps do (for comparison; they write c rows per tile).
bool iv_corrf_walk() {
  static const bool on = [] {
    const char* e = getenv("LP_IV_CORRF_WALK");
    return e && strcmp(e, "1") == 0;
  }();
  return on;
}

// Workgroups per interval of an interval-resident sweep: enough for about
// iv_target() workgroups in all (a few per resident slot), each walking
// ntiles / groups batch tiles; LP_IV_WG overrides the target.
int iv_target(int q) {
  static const int env = [] {
    const char* e = getenv("LP_IV_WG");
    return e ? atoi(e) : 0;
  }();
  if (env > 0) return env;
  return q == 64 ? 2048 : 1 << 30;
}

int iv_groups(int q, int ntiles, long Nc) {
  const long g = (iv_target(q) + Nc - 1) / Nc;
  return (int)std::max<long>(1, std::min<long>(ntiles, g));
}

template <int Q>
hipError_t sweep(int dir, const SweepArgs& a, hipStream_t st, int* partials) {
  constexpr int W4 = SWEEP_WAVES, EX = SWEEP_EX;
  const long Nc = a.Nl / a.c;
  if (Nc > 65535) return hipErrorNotSupported;  // intervals index the grid's y dimension
  const int ntiles = (a.B + EX * W4 - 1) / (EX * W4);
  const dim3 grid(ntiles, (unsigned)Nc);
  // Interval-resident kernels: every sweep at width 32; at width 64 (four layers,
  // 70 KB of LDS per workgroup) every sweep but the coarse levels' adjoint FRES
  // (iv_fres64). C-point storage (a.cpt, finest level) has interval-resident
  // kernels only.
  if constexpr (Q == 32 || Q == 64) {
    if (a.cpt && a.c != IV_CF) return hipErrorNotSupported;
    if (a.c == IV_CF &&
        (a.cpt || (iv_enabled() && (iv_fres64() > (a.G ? 1 : 0) ||
                                     !(Q == 64 && dir == DIR_ADJ && a.mode == SWEEP_FRES))))) {
      const int tg = a.mode == SWEEP_CORRF && !iv_corrf_walk() ? ntiles : iv_groups(Q, ntiles, Nc);
      const dim3 gi(tg, (unsigned)Nc);
      if (partials) *partials = (int)(gi.x * gi.y);
      // the next tile's rows are prefetched on the finest level only: with the
      // right-hand-side rows of a coarse level they would cost half the occupancy
      if (tg == ntiles) {
        if (a.G) sweep_iv<Q, true, 0>(dir, a, gi, st);
        else sweep_iv<Q, false, 0>(dir, a, gi, st);
      } else {
        if (a.G) sweep_iv<Q, true, 1>(dir, a, gi, st);
        else sweep_iv<Q, false, 2>(dir, a, gi, st);
      }
      return hipGetLastError();
    }
  }
  if (partials) *partials = (int)(grid.x * grid.y);
  const bool rec = a.dsig != nullptr;
  if (dir == DIR_FWD) {
    // only the final F-relaxation writes the sigma' record
    if (a.mode == SWEEP_FC) launch(k_fwd<Q, SWEEP_FC, W4, EX, false>, grid, 64 * W4, 0, st, a);
    else if (a.mode == SWEEP_FRES) launch(k_fwd<Q, SWEEP_FRES, W4, EX, false>, grid, 64 * W4, 0, st, a);
    else if (rec) launch(k_fwd<Q, SWEEP_CORRF, W4, EX, true>, grid, 64 * W4, 0, st, a);
    else launch(k_fwd<Q, SWEEP_CORRF, W4, EX, false>, grid, 64 * W4, 0, st, a);
  } else if (rec) {
    if (a.mode == SWEEP_FC) launch(k_adj<Q, SWEEP_FC, W4, EX, true>, grid, 64 * W4, 0, st, a);
    else if (a.mode == SWEEP_FRES) launch(k_adj<Q, SWEEP_FRES, W4, EX, true>, grid, 64 * W4, 0, st, a);
    else launch(k_adj<Q, SWEEP_CORRF, W4, EX, true>, grid, 64 * W4, 0, st, a);
  } else {
    if (a.mode == SWEEP_FC) launch(k_adj<Q, SWEEP_FC, W4, EX, false>, grid, 64 * W4, 0, st, a);
    else if (a.mode == SWEEP_FRES) launch(k_adj<Q, SWEEP_FRES, W4, EX, false>, grid, 64 * W4, 0, st, a);
    else launch(k_adj<Q, SWEEP_CORRF, W4, EX, false>, grid, 64 * W4, 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace mfma

bool mfma_width_supported(int q) { return q == 32 || q == 64; }

hipError_t mfma_sweep(int q, int dir, const SweepArgs& a, hipStream_t st, int* partials) {
  if (q == 32) return mfma::sweep<32>(dir, a, st, partials);
  if (q == 64) return mfma::sweep<64>(dir, a, st, partials);
  return hipErrorNotSupported;
}

hipError_t mfma_grad(int q, const GradArgs& a, hipStream_t st) {
  if (q == 32) return mfma::grad<32>(a, st);
  if (q == 64) return mfma::grad<64>(a, st);
  return hipErrorNotSupported;
}

hipError_t mfma_expand(int q, int act, const void* K, const void* b, const void* Uc, void* Y, int B, long k0,
                       long nk, double h, hipStream_t st) {
  if (nk <= 0 || B <= 0) return hipSuccess;
  if (nk > 65535) return hipErrorNotSupported;
  const dim3 grid((unsigned)((B + 63) / 64), (unsigned)nk);
  const float* Kp = static_cast<const float*>(K);
  const float* bp = static_cast<const float*>(b);
  const float* up = static_cast<const float*>(Uc);
  float* yp = static_cast<float*>(Y);
  if (q == 32) launch(mfma::k_expand<32>, grid, 256, 0, st, Kp, bp, up, yp, B, k0, (float)h, act);
  else if (q == 64) launch(mfma::k_expand<64>, grid, 256, 0, st, Kp, bp, up, yp, B, k0, (float)h, act);
  else return hipErrorNotSupported;
  return hipGetLastError();
}

hipError_t mfma_grad_partials(int q, const GradArgs& a, long nl, hipStream_t st) {
  if (q == 32) return mfma::grad_partials<32>(a, nl, st);
  if (q == 64) return mfma::grad_partials<64>(a, nl, st);
  return hipErrorNotSupported;
}

hipError_t mfma_grad_finish(int q, const GradArgs& a, hipStream_t st) {
  if (q == 32) return mfma::grad_finish<32>(a, st);
  if (q == 64) return mfma::grad_finish<64>(a, st);
  return hipErrorNotSupported;
}

}  // namespace lp
