// Residual norms of fp32 dense layers of width 32 or 64 on the matrix cores.
//
// State: r = u^n + h sigma(K_n u^n + b_n) - u^{n+1}; adjoint:
// r = lam^{n+1} + h K_n^T (sigma'(K_n u^n + b_n) * lam^{n+1}) - lam^n. A workgroup takes
// 64 examples (a wave 16) through a run of consecutive layers, so that a layer's
// output row is the next one's input and is read once; the next layer's weights and
// rows are requested before the current products, and LDS holds two layers. The
// arithmetic of a step is that of the sweeps and serial solves, but for tanh.
//
// One thread per example evaluated all Q activations and Q^2 products in a row and
// read every row twice. 512 layers of width 64, 4096 examples (0.54 GB of states), tanh,
// with the reduction and the read-back: state 562 us then, 245 now; adjoint 904 and 392
// (ReLU 471 and 196, 793 and 329). The state's rows are read once at 2.2 TB/s with
// tanh, 2.7 with ReLU: bound by the vector ALU, then by the fp32 matrix rate.
#include <algorithm>

#include "lp_dense_tile.h"

namespace lp {
namespace mfma {
namespace {

constexpr int RW = 4;  // waves per workgroup

// sigma (or sigma') of every value with the device library's tanh: the residual
// measures the solves, whose tanh has an absolute error of a few ulp of 1 (and so a
// relative one of percents for |z| near 1e-6).
template <typename V, int NB, int NV, bool DERIV>
__device__ __forceinline__ void apply_exact(V (&z)[NB], int act) {
  if (act != ACT_TANH) {
    apply<V, NB, NV>(z, act, DERIV);
    return;
  }
#pragma unroll
  for (int mb = 0; mb < NB; ++mb)
#pragma unroll
    for (int r = 0; r < NV; ++r) z[mb][r] = DERIV ? dact_f<float, ACT_TANH>(z[mb][r]) : act_f<float, ACT_TANH>(z[mb][r]);
}

// Adjoint, width 64: its rows and column operands are held to three waves per SIMD.
template <int Q, int DIR>
__global__ __launch_bounds__(64 * RW)
__attribute__((amdgpu_waves_per_eu(Q == 64 ? (DIR == DIR_FWD ? 4 : 3) : 4, 8)))
void k_resid(ResidArgs a, int ntiles, int run) {
  using C = Cfg<Q, RW>;
  using Lt = Lay<Q, 16>;
  using V = typename Lt::V;
  constexpr int NB = Lt::NB, NV = Lt::NV;
  constexpr bool FWD = DIR == DIR_FWD;
  __shared__ float W[2][C::WSZ];
  __shared__ double red[RW];
  const int lane = threadIdx.x & 63;
  const int tile = blockIdx.x % ntiles, g = blockIdx.x / ntiles;
  const int e = (tile * RW + (threadIdx.x >> 6)) * 16 + (lane & 15);
  const bool on = e < a.B;
  const size_t slice = (size_t)a.B * Q;
  const size_t row = (size_t)(on ? e : 0) * Q + 4 * (lane >> 4);
  const float* K = static_cast<const float*>(a.K);
  const float* bb = static_cast<const float*>(a.b);
  const float* U = static_cast<const float*>(a.U);
  const float* L = static_cast<const float*>(a.Lam);
  const float h = (float)a.h;
  // layers n0 .. n1 - 1: upwards for the state, downwards for the adjoint
  const int n0 = g * run, n1 = min(n0 + run, a.N), cnt = n1 - n0;
  auto layer = [&](int j) { return (size_t)(FWD ? n0 + j : n1 - 1 - j); };

  WRegs<Q, RW> wr;
  w_fetch<Q, RW>(wr, K, bb, layer(0));
  // x: the row that the step starts from; y: the row that its result is compared
  // with; u: the state that an adjoint step is linearised at
  V x[NB], y[NB], u[FWD ? 1 : NB];
  Lt::load(x, (FWD ? U : L) + (layer(0) + (FWD ? 0 : 1)) * slice + row);
  if constexpr (!FWD) Lt::load(u, U + layer(0) * slice + row);
  w_put<Q, RW>(W[0], wr);
  __syncthreads();
  double acc = 0.0;
  for (int j = 0; j < cnt; ++j) {
    const size_t n = layer(j), nn = layer(min(j + 1, cnt - 1));
    w_fetch<Q, RW>(wr, K, bb, nn);
    Lt::load(y, (FWD ? U + (n + 1) * slice : L + n * slice) + row);
    V s[NB];
    if constexpr (FWD) {
      Lt::template prod<C::LD>(s, x, W[j & 1], lane);
      apply_exact<V, NB, NV, false>(s, a.act);
    } else {
      V d[NB];
      Lt::template prod<C::LD, false>(d, u, W[j & 1], lane);
      Lt::load(u, U + nn * slice + row);
      apply_exact<V, NB, NV, true>(d, a.act);
#pragma unroll
      for (int mb = 0; mb < NB; ++mb) d[mb] = d[mb] * x[mb];
      Lt::template prod_t<C::LD, false>(s, d, W[j & 1], lane);
    }
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) {
      s[mb] = x[mb] + h * s[mb];
      x[mb] = y[mb];
    }
    if (on) acc += sq_diff<V, NB, NV>(s, y);
    w_put<Q, RW>(W[(j + 1) & 1], wr);
    __syncthreads();
  }
  const double s = wg_sum<RW>(acc, red);
  if (threadIdx.x == 0) a.partial[blockIdx.x] = s;
}

// Layers per workgroup: as many as leave about 4096 workgroups (four or more on each
// CU, in a few turns), at most 8, where the extra row and the first wait are an
// eighth of a run's.
template <int Q>
hipError_t resid(int dir, const ResidArgs& a, hipStream_t st, int* partials) {
  const int ntiles = (a.B + 16 * RW - 1) / (16 * RW);
  const int run = (int)std::clamp<long>((long)ntiles * a.N / 4096, 1, 8);
  const long grid = (long)ntiles * ((a.N + run - 1) / run);
  if (grid > 0x7fffffffL) return hipErrorNotSupported;
  if (partials) *partials = (int)grid;
  if (grid == 0) return hipSuccess;
  if (dir == DIR_FWD) launch(k_resid<Q, DIR_FWD>, dim3((unsigned)grid), 64 * RW, 0, st, a, ntiles, run);
  else launch(k_resid<Q, DIR_ADJ>, dim3((unsigned)grid), 64 * RW, 0, st, a, ntiles, run);
  return hipGetLastError();
}

}  // namespace
}  // namespace mfma

hipError_t mfma_resid(int q, int dir, const ResidArgs& a, hipStream_t st, int* partials) {
  if (q == 32) return mfma::resid<32>(dir, a, st, partials);
  if (q == 64) return mfma::resid<64>(dir, a, st, partials);
  return hipErrorNotSupported;
}

}  // namespace lp
