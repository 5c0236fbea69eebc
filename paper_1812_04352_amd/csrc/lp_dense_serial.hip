// Serial solves of fp32 dense layers of width 32 or 64 on the matrix cores: the
// coarsest level, the layer-serial trainer and evaluation.
//
// One wave per 16 examples runs through all N_l steps in order, so with a small
// batch there are few waves and the time per step is one wave's latency. Each
// weight is used by one lane of a wave, in one product, so it goes from L1/L2
// straight to the register that the matrix instruction reads; there is no LDS and
// no barrier (with many waves per CU the weights go through LDS, below). Through LDS,
// written at the end of the step before and read back at the start of the step, a
// step of width 32 took about 1300 cycles, of which its 16 matrix instructions take
// 512; 256 layers, 64 examples with opening and accuracy: 158 us before, 122 us now.
// The operands of the next SER_D steps and their right-hand-side, sigma' record or
// primal rows are in flight in register rings; every prefetch is issued
// unconditionally with its index clamped to valid rows, so the number of loads in
// flight is fixed and the waits stay exact. The arithmetic of a step, with the
// order of its sums, is that of the interval kernels.
#include "lp_dense_tile.h"

namespace lp {
namespace mfma {
namespace {

constexpr int MODE_SERIAL = 3;  // SweepArgs.mode of a whole-level serial solve

// Steps in flight: four at width 32. At width 64 a layer's operands take 80
// registers per lane forward and 64 transposed: two layers.
template <int Q>
constexpr int SER_D = Q <= 32 ? 4 : 2;

// Operands of z = K_n v + b_n, as Lay<Q, 16>::prod reads them from LDS: lane
// l = 16 g + i has K[16 ob + i][16 ib + 4 g ..] and b[16 ob + 4 g ..].
template <int Q>
struct FwdOps {
  static constexpr int NB = Q / 16;
  f32x4 a[NB][NB], b[NB];
  __device__ void fetch(const float* __restrict__ K, const float* __restrict__ bb, size_t n, int lane) {
    const int g = lane >> 4, i = lane & 15;
    const float* Kn = K + n * (size_t)(Q * Q) + i * Q + 4 * g;
    const float* bn = bb + n * (size_t)Q + 4 * g;
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
      b[ob] = *reinterpret_cast<const f32x4g*>(bn + 16 * ob);
#pragma unroll
      for (int ib = 0; ib < NB; ++ib) a[ob][ib] = *reinterpret_cast<const f32x4g*>(Kn + 16 * ob * Q + 16 * ib);
    }
  }
  // the blocks' chains of instructions in turn
  __device__ void prod(f32x4 (&z)[NB], const f32x4 (&v)[NB]) const {
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) z[ob] = b[ob];
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ob = 0; ob < NB; ++ob)
          z[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ob][ib][r], v[ib][r], z[ob], 0, 0, 0);
  }
};

// Operands of w = K_n^T s (Lay<Q, 16>::prod_t): K[16 ib + 4 g + r][16 ob + i].
template <int Q>
struct AdjOps {
  static constexpr int NB = Q / 16;
  float a[NB][NB][4];
  __device__ void fetch(const float* __restrict__ K, size_t n, int lane) {
    const int g = lane >> 4, i = lane & 15;
    const float* Kn = K + n * (size_t)(Q * Q) + 4 * g * Q + i;
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ob = 0; ob < NB; ++ob) a[ob][ib][r] = Kn[(16 * ib + r) * Q + 16 * ob];
  }
  __device__ void prod(f32x4 (&w)[NB], const f32x4 (&s)[NB]) const {
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) w[ob] = 0.f;
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ob = 0; ob < NB; ++ob)
          w[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ob][ib][r], s[ib][r], w[ob], 0, 0, 0);
  }
};

// Forward: U[j+1] = U[j] + h_l sigma(K_j U[j] + b_j) (+ G[j+1]), j = 0 .. N_l - 1;
// with REC the level-0 solve records sigma'(z) of every layer.
// (Two waves per SIMD are asked for where 256 registers suffice: the compiler then
// keeps the accumulators out of the accumulation registers.)
template <int Q, bool REC>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_ser_fwd(SweepArgs a) {
  using Lt = Lay<Q, 16>;
  using V = typename Lt::V;
  constexpr int NB = Lt::NB, NV = Lt::NV, D = SER_D<Q>;
  const int lane = threadIdx.x & 63;
  const int e = blockIdx.x * 16 + (lane & 15);
  const bool on = e < a.B;
  const size_t slice = (size_t)a.B * Q;
  const size_t row = (size_t)(on ? e : 0) * Q + 4 * (lane >> 4);
  const float* K = static_cast<const float*>(a.K);
  const float* bb = static_cast<const float*>(a.b);
  float* X = static_cast<float*>(a.X);
  const float* G = static_cast<const float*>(a.G);
  const int Nl = a.Nl;
  const float hl = (float)a.hl;

  // rings: slot u holds layer j and G row j + 1 for the step j = u (mod D)
  FwdOps<Q> op[D];
  V gr[D][NB];
#pragma unroll
  for (int u = 0; u < D; ++u) op[u].fetch(K, bb, (size_t)min(u, Nl - 1) * a.stride, lane);
  if (G) {
#pragma unroll
    for (int u = 0; u < D; ++u) Lt::load(gr[u], G + (size_t)min(u + 1, Nl) * slice + row);
  }
  V v[NB];
#pragma unroll
  for (int mb = 0; mb < NB; ++mb) v[mb] = 0.f;
  if (on) Lt::load(v, X + row);
  for (int j0 = 0; j0 < Nl; j0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int j = j0 + u;
      if (j >= Nl) break;
      V s[NB];
      op[u].prod(s, v);
      op[u].fetch(K, bb, (size_t)min(j + D, Nl - 1) * a.stride, lane);
      if constexpr (REC) {
        V dz[NB];
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) dz[mb] = s[mb];
        apply<V, NB, NV>(dz, a.act, true);
        store_dsig<Lt>(a.dsig, (size_t)j * a.stride * slice + row, a.act, dz, on);
      }
      apply<V, NB, NV>(s, a.act, false);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = v[mb] + hl * s[mb];
      if (G) {
        add_to<V, NB>(v, gr[u]);
        Lt::load(gr[u], G + (size_t)min(j + 1 + D, Nl) * slice + row);
      }
      if (on) Lt::store(X + (size_t)(j + 1) * slice + row, v);
    }
  }
}

// Adjoint: Lam[i] = Lam[i+1] + h_l K_i^T (sigma'(K_i U_f[i] + b_i) * Lam[i+1]) (+ G[i]),
// i = N_l - 1 .. 0, the primal state (row i * ustride of Uf, or the record at fine
// index i * stride, RK = 1 bits, 2 fp32).
template <int Q, int RK>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(RK == 0 ? 1 : 2, 8))) void k_ser_adj(SweepArgs a) {
  using Lt = Lay<Q, 16>;
  using V = typename Lt::V;
  constexpr bool REC = RK != 0;
  constexpr int NB = Lt::NB, NV = Lt::NV, D = SER_D<Q>;
  const int lane = threadIdx.x & 63;
  const int e = blockIdx.x * 16 + (lane & 15);
  const bool on = e < a.B;
  const size_t slice = (size_t)a.B * Q;
  const size_t row = (size_t)(on ? e : 0) * Q + 4 * (lane >> 4);
  const float* K = static_cast<const float*>(a.K);
  const float* bb = static_cast<const float*>(a.b);
  const float* Uf = static_cast<const float*>(a.Uf);
  float* X = static_cast<float*>(a.X);
  const float* G = static_cast<const float*>(a.G);
  const int Nl = a.Nl;
  const float hl = (float)a.hl;

  // rings, slot u for the step j = u (mod D), i = Nl - 1 - j: layer i, and the record
  // (or primal) and G rows of the step
  AdjOps<Q> op[D];
  FwdOps<Q> fo[REC ? 1 : D];
  RecRow<Lt, RK == 1> rr[REC ? D : 1];
  V ur[REC ? 1 : D][NB], gr[D][NB];
#pragma unroll
  for (int u = 0; u < D; ++u) {
    const int i = max(Nl - 1 - u, 0);  // every lane reads a valid row
    op[u].fetch(K, (size_t)i * a.stride, lane);
    if constexpr (REC) {
      rr[u].load(a.dsig, (size_t)i * a.stride * slice + row);
    } else {
      fo[u].fetch(K, bb, (size_t)i * a.stride, lane);
      Lt::load(ur[u], Uf + (size_t)i * a.ustride * slice + row);
    }
    if (G) Lt::load(gr[u], G + (size_t)i * slice + row);
  }
  V v[NB];
#pragma unroll
  for (int mb = 0; mb < NB; ++mb) v[mb] = 0.f;
  if (on) Lt::load(v, X + (size_t)Nl * slice + row);
  for (int j0 = 0; j0 < Nl; j0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int j = j0 + u;
      if (j >= Nl) break;
      const int i = Nl - 1 - j, ip = max(i - D, 0);
      V d[NB], w[NB];
      if constexpr (REC) {
        rr[u].get(d);
        rr[u].load(a.dsig, (size_t)ip * a.stride * slice + row);
      } else {
        fo[u].prod(d, ur[u]);
        fo[u].fetch(K, bb, (size_t)ip * a.stride, lane);
        apply<V, NB, NV>(d, a.act, true);
        Lt::load(ur[u], Uf + (size_t)ip * a.ustride * slice + row);
      }
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) d[mb] = d[mb] * v[mb];
      op[u].prod(w, d);
      op[u].fetch(K, (size_t)ip * a.stride, lane);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = v[mb] + hl * w[mb];
      if (G) {
        add_to<V, NB>(v, gr[u]);
        Lt::load(gr[u], G + (size_t)ip * slice + row);
      }
      if (on) Lt::store(X + (size_t)i * slice + row, v);
    }
  }
}

// ------------------------------------------------------------------ many waves
// With several waves on each CU the direct loads (16 rows of 64 bytes an instruction)
// are bound by the caches. Here a wave fetches a layer in memory order and turns it
// round through LDS (double buffer, one wave: program order suffices, the barriers
// are nominal). The layer after next is on its way in registers.

template <int Q, bool REC>
__global__ __launch_bounds__(64) void k_ser_fwd_lds(SweepArgs a) {
  using C = Cfg<Q, 1>;
  using Lt = Lay<Q, 16>;
  using V = typename Lt::V;
  constexpr int NB = Lt::NB, NV = Lt::NV, D = SER_D<Q>;
  __shared__ float W[2][C::WSZ];
  const int lane = threadIdx.x & 63;
  const int e = blockIdx.x * 16 + (lane & 15);
  const bool on = e < a.B;
  const size_t slice = (size_t)a.B * Q;
  const size_t row = (size_t)(on ? e : 0) * Q + 4 * (lane >> 4);
  const float* K = static_cast<const float*>(a.K);
  const float* bb = static_cast<const float*>(a.b);
  float* X = static_cast<float*>(a.X);
  const float* G = static_cast<const float*>(a.G);
  const int Nl = a.Nl;
  const float hl = (float)a.hl;

  // rings: slot u holds layer j+1's weights and G row j+1 for the step j = u (mod D)
  WRegs<Q, 1> wr[D];
  V gr[D][NB];
  {
    WRegs<Q, 1> w0;
    w_fetch<Q, 1>(w0, K, bb, 0);
    // every prefetch is issued unconditionally (indices clamped to valid rows), so
    // the number of loads in flight is fixed and the waits stay exact
#pragma unroll
    for (int u = 0; u < D; ++u) w_fetch<Q, 1>(wr[u], K, bb, (size_t)min(u + 1, Nl - 1) * a.stride);
    if (G) {
#pragma unroll
      for (int u = 0; u < D; ++u) Lt::load(gr[u], G + (size_t)min(u + 1, Nl) * slice + row);  // valid rows
    }
    w_put<Q, 1>(W[0], w0);
  }
  V v[NB];
#pragma unroll
  for (int mb = 0; mb < NB; ++mb) v[mb] = 0.f;
  if (on) Lt::load(v, X + row);
  __syncthreads();
  for (int j0 = 0; j0 < Nl; j0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int j = j0 + u;
      if (j >= Nl) break;
      V s[NB];
      Lt::template prod<C::LD>(s, v, W[j & 1], lane);
      if constexpr (REC) {
        V dz[NB];
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) dz[mb] = s[mb];
        apply<V, NB, NV>(dz, a.act, true);
        store_dsig<Lt>(a.dsig, (size_t)j * a.stride * slice + row, a.act, dz, on);
      }
      apply<V, NB, NV>(s, a.act, false);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = v[mb] + hl * s[mb];
      if (G) {
        add_to<V, NB>(v, gr[u]);
        Lt::load(gr[u], G + (size_t)min(j + 1 + D, Nl) * slice + row);
      }
      if (on) Lt::store(X + (size_t)(j + 1) * slice + row, v);
      // after the last step this writes a layer nobody reads
      w_put<Q, 1>(W[(j + 1) & 1], wr[u]);
      w_fetch<Q, 1>(wr[u], K, bb, (size_t)min(j + 1 + D, Nl - 1) * a.stride);
      __syncthreads();
    }
  }
}

template <int Q, int RK>
__global__ __launch_bounds__(64) void k_ser_adj_lds(SweepArgs a) {
  using C = Cfg<Q, 1>;
  using Lt = Lay<Q, 16>;
  using V = typename Lt::V;
  constexpr int NB = Lt::NB, NV = Lt::NV, D = SER_D<Q>;
  constexpr bool REC = RK != 0;
  __shared__ float W[2][C::WSZ];
  const int lane = threadIdx.x & 63;
  const int e = blockIdx.x * 16 + (lane & 15);
  const bool on = e < a.B;
  const size_t slice = (size_t)a.B * Q;
  const size_t row = (size_t)(on ? e : 0) * Q + 4 * (lane >> 4);
  const float* K = static_cast<const float*>(a.K);
  const float* bb = static_cast<const float*>(a.b);
  const float* Uf = static_cast<const float*>(a.Uf);
  float* X = static_cast<float*>(a.X);
  const float* G = static_cast<const float*>(a.G);
  const int Nl = a.Nl;
  const float hl = (float)a.hl;

  // rings, slot u for the step j = u (mod D), i = Nl - 1 - j: the weights of the
  // next step's layer i - 1, and the step's own record (or primal) and G rows
  WRegs<Q, 1> wr[D];
  RecRow<Lt, RK == 1> rr[REC ? D : 1];
  V ur[REC ? 1 : D][NB], gr[D][NB];
  {
    WRegs<Q, 1> w0;
    w_fetch<Q, 1>(w0, K, bb, (size_t)(Nl - 1) * a.stride);
    // every prefetch is issued unconditionally (indices clamped to valid rows), so
    // the number of loads in flight is fixed and the waits stay exact
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int i = max(Nl - 1 - u, 0);  // every lane reads a valid row
      w_fetch<Q, 1>(wr[u], K, bb, (size_t)max(i - 1, 0) * a.stride);
      if constexpr (REC) rr[u].load(a.dsig, (size_t)i * a.stride * slice + row);
      else Lt::load(ur[u], Uf + (size_t)i * a.ustride * slice + row);
      if (G) Lt::load(gr[u], G + (size_t)i * slice + row);
    }
    w_put<Q, 1>(W[0], w0);
  }
  V v[NB];
#pragma unroll
  for (int mb = 0; mb < NB; ++mb) v[mb] = 0.f;
  if (on) Lt::load(v, X + (size_t)Nl * slice + row);
  __syncthreads();
  for (int j0 = 0; j0 < Nl; j0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int j = j0 + u;
      if (j >= Nl) break;
      const int i = Nl - 1 - j;
      const float* Wj = W[j & 1];
      V d[NB], w[NB];
      const int ip = max(i - D, 0);
      if constexpr (REC) {
        rr[u].get(d);
        rr[u].load(a.dsig, (size_t)ip * a.stride * slice + row);
      } else {
        Lt::template prod<C::LD>(d, ur[u], Wj, lane);
        apply<V, NB, NV>(d, a.act, true);
        Lt::load(ur[u], Uf + (size_t)ip * a.ustride * slice + row);
      }
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) d[mb] = d[mb] * v[mb];
      Lt::template prod_t<C::LD>(w, d, Wj, lane);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) v[mb] = v[mb] + hl * w[mb];
      if (G) {
        add_to<V, NB>(v, gr[u]);
        Lt::load(gr[u], G + (size_t)ip * slice + row);
      }
      if (on) Lt::store(X + (size_t)i * slice + row, v);
      // after the last step this writes a layer nobody reads
      w_put<Q, 1>(W[(j + 1) & 1], wr[u]);
      w_fetch<Q, 1>(wr[u], K, bb, (size_t)max(i - 1 - D, 0) * a.stride);
      __syncthreads();
    }
  }
}

template <int Q>
hipError_t serial(int dir, const SerialArgs& s, hipStream_t st) {
  SweepArgs a{};
  a.act = s.act;
  a.mode = MODE_SERIAL;
  a.K = s.K;
  a.b = s.b;
  a.Uf = s.Uf;
  a.B = s.B;
  a.Nl = s.Nl;
  a.c = 1;
  a.stride = s.stride;
  a.hl = s.hl;
  a.X = s.X;
  a.G = s.G;
  a.dsig = s.dsig;
  a.ustride = s.ustride;
  const dim3 grid((s.B + 15) / 16, 1);
  // Direct loads up to one wave per CU at width 64 and two at width 32, and at width 64 not
  // where a step needs more registers than they leave (a recorded forward step, an adjoint
  // step with both products). 128 layers, us, direct / through LDS, ReLU:
  //   width 32, 500 and 8192 examples: forward 56 / 75 and 67 / 85, with record 94 / 113
  //     and 99 / 120, adjoint with record 67 / 79 and 73 / 87, without 108 / 116 and
  //     114 / 121; 256 layers, 16384 examples: forward 255 / 227
  //   width 64, 500 and 4096 examples: forward 176 / 192 and 185 / 201, adjoint with record
  //     188 / 214 and 193 / 220; not chosen: forward with record 256 / 245 and 259 / 253,
  //     adjoint without 328 / 321 and 330 / 325; 256 layers, 16384 examples: forward 690 / 543
  const bool direct = s.B <= (Q == 64 ? 4096 : 8192);
  if (dir == DIR_FWD) {
    if (s.dsig) {
      if constexpr (Q != 64) {
        if (direct) {
          launch(k_ser_fwd<Q, true>, grid, 64, 0, st, a);
          return hipGetLastError();
        }
      }
      launch(k_ser_fwd_lds<Q, true>, grid, 64, 0, st, a);
    } else if (direct) {
      launch(k_ser_fwd<Q, false>, grid, 64, 0, st, a);
    } else {
      launch(k_ser_fwd_lds<Q, false>, grid, 64, 0, st, a);
    }
  } else if (!s.dsig) {
    if constexpr (Q != 64) {
      if (direct) {
        launch(k_ser_adj<Q, 0>, grid, 64, 0, st, a);
        return hipGetLastError();
      }
    }
    launch(k_ser_adj_lds<Q, 0>, grid, 64, 0, st, a);
  } else if (s.act == ACT_RELU) {
    if (direct) launch(k_ser_adj<Q, 1>, grid, 64, 0, st, a);
    else launch(k_ser_adj_lds<Q, 1>, grid, 64, 0, st, a);
  } else {
    if (direct) launch(k_ser_adj<Q, 2>, grid, 64, 0, st, a);
    else launch(k_ser_adj_lds<Q, 2>, grid, 64, 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace
}  // namespace mfma

hipError_t mfma_serial(int q, int dir, const SerialArgs& a, hipStream_t st) {
  if (q == 32) return mfma::serial<32>(dir, a, st);
  if (q == 64) return mfma::serial<64>(dir, a, st);
  return hipErrorNotSupported;
}

}  // namespace lp
