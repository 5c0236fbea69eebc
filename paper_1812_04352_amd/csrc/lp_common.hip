// Kernels shared by every layer family: row copies (the MGRIT cold start), the
// fixed-order residual-norm reduction, and the boundary helpers of the network
// (opening layer and its gradient, the plain gradient step). The helpers sit
// outside the per-iteration hot path. The loss helper lives in lp_loss.hip.
#include <math.h>

#include <algorithm>
#include <limits>
#include <type_traits>

#include "lp_device.h"
#include "lp_internal.h"
#include "lp_open_geo.h"

namespace lp {
namespace {

constexpr int NT = 256;

// X[dst_row0 + t*dst_step] = X[src_row] for t = 0..count-1 (16-byte units; the
// source row is not among the destinations). Workgroup row blockIdx.y takes
// destination rows rows * blockIdx.y .. + rows - 1: each thread reads its units
// of the source row once and writes them to those rows.
__global__ __launch_bounds__(NT) void k_copy_rows(uint4* X, size_t units, long src_row,
                                                  long dst_row0, long dst_step, long count, long rows) {
  const long t0 = (long)blockIdx.y * rows, t1 = min(count, t0 + rows);
  for (size_t u = (size_t)blockIdx.x * NT + threadIdx.x; u < units; u += (size_t)gridDim.x * NT) {
    const uint4 v = X[(size_t)src_row * units + u];
    for (long t = t0; t < t1; ++t) X[(size_t)(dst_row0 + t * dst_step) * units + u] = v;
  }
}

// Sticky per-device record of a non-finite residual norm (any MGRIT solve or
// residual-norm call on this device since the flag was last cleared). Set by the
// reduction below with an ordinary global store; read and cleared by
// lp_check_finite.
__device__ uint32_t g_nonfinite = 0u;

// out[0] = sqrt(sum of partial[0..n)), summed in a fixed order: thread t adds
// partial[t], partial[t + NTR], ... in index order (eight loads issued at a time,
// so the serial chain waits once per eight), then the workgroup tree.
constexpr int NTR = 1024;
__global__ __launch_bounds__(NTR) void k_norm_reduce(const double* partial, int n, double* out) {
  __shared__ double sh[NTR];
  double s = 0.0;
  int i = threadIdx.x;
  for (; i + 7 * NTR < n; i += 8 * NTR) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = partial[i + k * NTR];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += v[k];
  }
  for (; i < n; i += NTR) s += partial[i];
  s = block_sum<NTR>(s, sh);
  if (threadIdx.x == 0) {
    const double r = sqrt(s);
    out[0] = r;
    if (!isfinite(r)) g_nonfinite = 1u;
  }
}

// dst[i] = src[i] over 16-byte units.
__global__ __launch_bounds__(NT) void k_copy16(uint4* dst, const uint4* src, size_t units) {
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < units; i += (size_t)gridDim.x * NT) dst[i] = src[i];
}

__global__ __launch_bounds__(NT) void k_zero(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT) p[i] = 0u;
}

unsigned grid_for(size_t work) {
  size_t g = (work + NT - 1) / NT;
  if (g > 65535u * 8u) g = 65535u * 8u;
  return (unsigned)(g ? g : 1);
}

// ---------------------------------------------------------------- opening layer

// u0[e][r] = sigma(sum_f L[r][f] y[e][f]), f in order. A workgroup owns a tile of
// OE examples x OR rows; both operands pass through LDS in pieces of OF features
// (coalesced loads, the next piece requested before the current one is used), and
// a thread sums a 2 x 2 patch of the tile from 16-byte LDS reads (row pitch OF + 4
// words: the 16 rows of a read start 4 banks apart). One thread per output, its
// two rows read from global memory feature by feature, measured 122 us for
// 16384 x 128 -> 32 fp32 (bound by uncoalesced reads and a serial chain of loads).
constexpr int OE = 32, OR = 32;
template <typename T> constexpr int OF = 512 / (int)sizeof(T);  // 512-byte pieces of a row

template <typename T, int ACT>
__global__ __launch_bounds__(NT) void k_open_dense(const T* y, const T* L, T* u0, int B, int q, int nf) {
  constexpr int F = OF<T>, LD = F + 16 / (int)sizeof(T), NLD = (OE + OR) * F / NT;
  __shared__ __align__(16) T sh[(OE + OR) * LD];
  const int e0 = blockIdx.x * OE, r0 = blockIdx.y * OR, t = threadIdx.x;
  // piece f0: rows 0 .. OE-1 of sh are the examples, the rest the weight rows; zero outside
  T reg[NLD];
  auto fetch = [&](int f0) {
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int i = t + k * NT, row = i / F, f = f0 + i % F;
      const bool in = f < nf && (row < OE ? e0 + row < B : r0 + row - OE < q);
      const T* p = row < OE ? y + (size_t)(e0 + row) * nf : L + (size_t)(r0 + row - OE) * nf;
      reg[k] = in ? p[f] : T(0);
    }
  };
  const int te = t % 16, tr = t / 16;
  T acc[2][2] = {{T(0), T(0)}, {T(0), T(0)}};
  fetch(0);
  for (int f0 = 0; f0 < nf; f0 += F) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int i = t + k * NT;
      sh[(i / F) * LD + i % F] = reg[k];
    }
    __syncthreads();
    if (f0 + F < nf) fetch(f0 + F);
    using V = typename Vec16<T>::type;
    constexpr int nv = Vec16<T>::n;
    const int nn = (min(F, nf - f0) + nv - 1) / nv;  // past nf both operands are zero
#pragma unroll 4
    for (int v = 0; v < nn; ++v) {
      V a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = *reinterpret_cast<const V*>(sh + (te + 16 * i) * LD + nv * v);
        b[i] = *reinterpret_cast<const V*>(sh + (OE + tr + 16 * i) * LD + nv * v);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if constexpr (nv == 4) {
            acc[i][j] = fma(b[j].x, a[i].x, acc[i][j]);
            acc[i][j] = fma(b[j].y, a[i].y, acc[i][j]);
            acc[i][j] = fma(b[j].z, a[i].z, acc[i][j]);
            acc[i][j] = fma(b[j].w, a[i].w, acc[i][j]);
          } else {
            acc[i][j] = fma(b[j].x, a[i].x, acc[i][j]);
            acc[i][j] = fma(b[j].y, a[i].y, acc[i][j]);
          }
        }
    }
  }
  // through LDS, so that the output rows are written in order
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) sh[(te + 16 * i) * (OR + 1) + tr + 16 * j] = act_f<T, ACT>(acc[i][j]);
  __syncthreads();
  for (int i = t; i < OE * OR; i += NT) {
    const int e = i / OR, r = i % OR;
    if (e0 + e < B && r0 + r < q) u0[(size_t)(e0 + e) * q + r0 + r] = sh[e * (OR + 1) + r];
  }
}

// u0[e][co][y][x] = sigma(sum_{ty,tx} L[co][0][ty][tx] y[e][0][y+ty-1][x+tx-1]), zero padded.
template <typename T, int ACT>
__global__ __launch_bounds__(NT) void k_open_conv(const T* y, const T* L, T* u0, int B, int C, int H, int W) {
  const size_t tot = (size_t)B * C * H * W;
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < tot; i += (size_t)gridDim.x * NT) {
    size_t t = i;
    const int x = (int)(t % W); t /= W;
    const int yy = (int)(t % H); t /= H;
    const int co = (int)(t % C);
    const size_t e = t / C;
    T acc = T(0);
    for (int ty = 0; ty < 3; ++ty) {
      const int sy = yy + ty - 1;
      if (sy < 0 || sy >= H) continue;
      for (int tx = 0; tx < 3; ++tx) {
        const int sx = x + tx - 1;
        if (sx < 0 || sx >= W) continue;
        acc = fma(L[co * 9 + ty * 3 + tx], y[e * H * W + (size_t)sy * W + sx], acc);
      }
    }
    u0[i] = act_f<T, ACT>(acc);
  }
}

// dL[r][f] = sum_e sigma'(z_er) lam0[e][r] y[e][f]; one workgroup of 8 or 16 waves
// per row r (there is no workspace to combine several in). Lane l of a wave holds the
// features l, l + 64, ... of GE examples at a time, read once, coalesced, straight
// into registers, the next GE requested before the current ones are used; the
// waves run without barriers. The GE values of z are added over the lanes in one
// butterfly that halves their number per exchange, so that sigma' runs once for
// all of them, and come back as scalars. fp32 sums over GE examples, then fp64 in
// a fixed order. ReLU's decision has to be that of the opening layer, which sums z
// feature by feature: where the two orders could fall on either side of zero (|z| below
// about nf / 2 eps sum |L y|: in fp32 one example in 20000 of 64 features, one in 1000
// of 1024), z is summed again in its order, from scalar loads. 16384 examples, 32 rows,
// fp32, us: 128 features tanh 1776 with a barrier and a chain of loads per 256
// examples, 156 now, ReLU 1497 and 176; 1024 features ReLU 9937 and 1091.
constexpr int GNT = 1024;

template <typename T>
__device__ __forceinline__ T lane_value(T v, int lane) {
  if constexpr (sizeof(T) == 4) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
  } else {
    const long long b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)b >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
  }
}

// FPL features per lane, GE examples (a power of two <= 8) in flight, WAVES waves
template <typename T, int ACT, int FPL, int GE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_open_grad_dense(const T* y, const T* L, const T* lam0, T* dL,
                                                                int B, int q, int nf) {
  __shared__ double sh[WAVES][64];
  const int r = blockIdx.x, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int LG = GE == 8 ? 3 : GE == 4 ? 2 : GE == 2 ? 1 : 0;
  T w[FPL];
  double acc[FPL];
#pragma unroll
  for (int k = 0; k < FPL; ++k) {
    const int f = lane + 64 * k;
    w[k] = f < nf ? L[(size_t)r * nf + f] : T(0);
    acc[k] = 0.0;
  }
  T yn[GE][FPL], ln;  // loads without a branch, past the end the last valid value again
  const int me = lane >> (6 - LG);  // the example whose z this lane ends up with
  auto fetch = [&](int e0) {
#pragma unroll
    for (int i = 0; i < GE; ++i)
#pragma unroll
      for (int k = 0; k < FPL; ++k) {
        const int f = lane + 64 * k;
        yn[i][k] = y[(size_t)min(e0 + i, B - 1) * nf + min(f, nf - 1)];
      }
    ln = lam0[(size_t)min(e0 + me, B - 1) * q + r];
  };
  // the sums of p[0 .. GE) over the lanes, that of example `me` in each lane
  auto lane_sums = [&](T(&p)[GE]) {
#pragma unroll
    for (int k = 0; k < LG; ++k) {
      const int half = GE >> (k + 1), off = 32 >> k;
      const bool up = lane & off;
#pragma unroll
      for (int i = 0; i < half; ++i) {
        // (a choice between the array's elements themselves would index it at run time)
        const T lo = p[i], hi = p[i + half], send = up ? lo : hi, keep = up ? hi : lo;
        p[i] = keep + __shfl_xor(send, off, 64);
      }
    }
#pragma unroll
    for (int k = LG; k < 6; ++k) p[0] += __shfl_xor(p[0], 32 >> k, 64);
    return p[0];
  };
  fetch(wave * GE);
  for (int e0 = wave * GE; e0 < B; e0 += WAVES * GE) {
    T v[GE][FPL], p[GE], m[GE];
    const T lam = ln;
#pragma unroll
    for (int i = 0; i < GE; ++i) {
      p[i] = m[i] = T(0);
#pragma unroll
      for (int k = 0; k < FPL; ++k) {
        v[i][k] = e0 + i < B && lane + 64 * k < nf ? yn[i][k] : T(0);
        p[i] = fma(w[k], v[i][k], p[i]);
        m[i] = fma(fabs(w[k]), fabs(v[i][k]), m[i]);  // ReLU only
      }
    }
    fetch(e0 + WAVES * GE);
    T z = lane_sums(p);
    if constexpr (ACT == ACT_RELU) {
      // each order's rounding: (nf + FPL + 6) / 2 eps sum |L y| together; first by a bound
      // of the sum that takes no exchange, 64 times the largest lane's part
      constexpr T eps = std::numeric_limits<T>::epsilon();
      const int c = (nf + FPL + 8) >> 1;
      const T zs = ldexp(fabs(z), std::numeric_limits<T>::digits - 1 - 6 - (32 - __builtin_clz(c)));
      uint64_t any = 0;
#pragma unroll
      for (int i = 0; i < GE; ++i) any |= __ballot(lane_value(zs, i << (6 - LG)) < m[i]);
      if (any) {
        const uint64_t near = __ballot(fabs(z) < T(c) * eps * lane_sums(m));
        for (int i = 0; i < GE; ++i) {
          if (!(near >> (i << (6 - LG)) & 1)) continue;  // past B: 0 < 0
          const T* yr = y + (size_t)(e0 + i) * nf;
          T zi = T(0);
#pragma unroll 8
          for (int f = 0; f < nf; ++f) zi = fma(L[(size_t)r * nf + f], yr[f], zi);
          z = me == i ? zi : z;
        }
      }
    }
    const T s = e0 + me < B ? dact_f<T, ACT>(z) * lam : T(0);
    T a[FPL];
#pragma unroll
    for (int i = 0; i < GE; ++i) {
      const T si = lane_value(s, i << (6 - LG));
#pragma unroll
      for (int k = 0; k < FPL; ++k) a[k] = i == 0 ? si * v[i][k] : fma(si, v[i][k], a[k]);
    }
#pragma unroll
    for (int k = 0; k < FPL; ++k) acc[k] += (double)a[k];
  }
#pragma unroll
  for (int k = 0; k < FPL; ++k) {
    __syncthreads();
    sh[wave][lane] = acc[k];
    __syncthreads();
    const int f = lane + 64 * k;
    if (wave == 0 && f < nf) {
      double t = 0.0;
      for (int j = 0; j < WAVES; ++j) t += sh[j][lane];
      dL[(size_t)r * nf + f] = (T)t;
    }
  }
}

// Up to 8 features: a thread takes an example, so that no lane is idle for want of
// features, and sums its z in the order of k_open_dense. NF >= nf; the loads of FE
// examples of a thread are issued together. 5000 examples of 2 features, fp64, 8 rows:
// a lane per feature 165 us, 13 so.
template <typename T, int ACT, int NF>
__global__ __launch_bounds__(GNT) void k_open_grad_few(const T* y, const T* L, const T* lam0, T* dL, int B, int q,
                                                       int nf) {
  constexpr int FE = 4, WAVES = GNT / 64;
  __shared__ double sh[WAVES][NF];
  const int r = blockIdx.x, t = threadIdx.x;
  T w[NF];
  double acc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    w[f] = f < nf ? L[(size_t)r * nf + f] : T(0);
    acc[f] = 0.0;
  }
  for (long e0 = t; e0 < B; e0 += FE * GNT) {
    T v[FE][NF], lam[FE];
#pragma unroll
    for (int i = 0; i < FE; ++i) {
      const long e = e0 + (long)i * GNT;
      lam[i] = e < B ? lam0[(size_t)e * q + r] : T(0);
#pragma unroll
      for (int f = 0; f < NF; ++f) v[i][f] = e < B && f < nf ? y[(size_t)e * nf + f] : T(0);
    }
#pragma unroll
    for (int i = 0; i < FE; ++i) {
      T z = T(0);
#pragma unroll
      for (int f = 0; f < NF; ++f) z = fma(w[f], v[i][f], z);
      const T s = dact_f<T, ACT>(z) * lam[i];
#pragma unroll
      for (int f = 0; f < NF; ++f) acc[f] += (double)(s * v[i][f]);
    }
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc[f] += __shfl_xor(acc[f], off, 64);
    if ((t & 63) == 0) sh[t >> 6][f] = acc[f];
  }
  __syncthreads();
  if (t < nf) {
    double a = 0.0;
    for (int k = 0; k < WAVES; ++k) a += sh[k][t];
    dL[(size_t)r * nf + t] = (T)a;
  }
}

template <typename T, int ACT>
void open_grad_dense(const T* y, const T* L, const T* lam0, T* dL, int B, int q, int nf, hipStream_t st) {
  const auto few = [&](auto n) {
    k_open_grad_few<T, ACT, decltype(n)::value><<<q, GNT, 0, st>>>(y, L, lam0, dL, B, q, nf);
  };
  // about 64 registers of examples in flight per lane; fp64 from two features a lane on
  // and fp32 with 16 take half the waves, with twice the registers each (at 16 waves they
  // spill: 1024 features, 16384 examples, 32 rows, tanh: fp64 12.4 ms, 3.1 with 8 waves;
  // fp32 2.9 ms and 1.0)
  const auto run = [&](auto fpl) {
    constexpr int FPL = decltype(fpl)::value, W = FPL * (int)sizeof(T) / 4;
    constexpr int GE = W <= 4 ? 8 : W <= 8 ? 4 : W <= 16 ? 2 : 1;
    constexpr int WAVES = W > 8 || (sizeof(T) == 8 && FPL > 1) ? 8 : 16;
    k_open_grad_dense<T, ACT, FPL, GE, WAVES><<<q, 64 * WAVES, 0, st>>>(y, L, lam0, dL, B, q, nf);
  };
  if (nf <= 2) few(std::integral_constant<int, 2>{});
  else if (nf <= 8) few(std::integral_constant<int, 8>{});
  else if (nf <= 64) run(std::integral_constant<int, 1>{});
  else if (nf <= 128) run(std::integral_constant<int, 2>{});
  else if (nf <= 256) run(std::integral_constant<int, 4>{});
  else if (nf <= 512) run(std::integral_constant<int, 8>{});
  else run(std::integral_constant<int, 16>{});
}

// dL[co][0][ty][tx] = sum_e sum_p sigma'(z[e,co,p]) lam0[e,co,p] y[e, p + t]: one
// workgroup of 1024 threads per weight (co, ty, tx) (there is no workspace to
// combine several in). Each recomputes its channel's z, so its work is that of the
// window reads and the activation. Groups of IM images (IM P <= OCP GNT pixels)
// pass through LDS with a zero halo, the next group's values requested before the
// current one is used; a thread's pixels lie at the same offsets in every group.
// fp32 sums over a thread's pixels of one group, then fp64 in a fixed order.
// 500 images of 28 x 28: 2245 us with one workgroup per channel and one pixel per
// thread straight from memory (a chain of loads), 179 us now.
using open_conv::OCP;
using open_conv::OC_LDS;
static_assert(open_conv::GNT == GNT, "threads of k_open_grad_conv");

template <int ACT>
__global__ __launch_bounds__(GNT) void k_open_grad_conv(const float* y, const float* L, const float* lam0, float* dL,
                                                        int B, int C, int H, int W) {
  __shared__ float img[OC_LDS];
  __shared__ double sh[GNT];
  const int co = blockIdx.x / 9, tap = blockIdx.x % 9, t = threadIdx.x;
  const open_conv::Group g = open_conv::group(H, W);
  const int P = g.P, PW = g.PW, IM = g.IM;
  float w[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) w[k] = L[co * 9 + k];
  for (int i = t; i < IM * g.PH; i += GNT) img[i] = 0.f;
  open_conv::Pixel px[OCP];
#pragma unroll
  for (int k = 0; k < OCP; ++k) px[k] = open_conv::pixel(g, W, C, co, t + k * GNT);
  const int toff = tap / 3 * PW + tap % 3;
  float yv[OCP], lv[OCP];
  auto fetch = [&](int e0) {
    const float* ye = y + (size_t)e0 * P;
    const float* le = lam0 + (size_t)e0 * C * P;
    const int n = open_conv::images(g, B, e0);
#pragma unroll
    for (int k = 0; k < OCP; ++k) {
      const bool in = open_conv::live(px[k], n);
      yv[k] = in ? ye[t + k * GNT] : 0.f;
      lv[k] = in ? le[px[k].gl] : 0.f;
    }
  };
  fetch(0);
  double acc = 0.0;
  for (int e0 = 0;; e0 += IM) {
    const int n = open_conv::images(g, B, e0);
    float lam[OCP];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < OCP; ++k) {
      lam[k] = lv[k];
      if (open_conv::stored(g, px[k])) img[open_conv::store_index(g, px[k])] = yv[k];
    }
    __syncthreads();
    if (B - e0 > IM) fetch(e0 + IM);
    float a = 0.f;
#pragma unroll
    for (int k = 0; k < OCP; ++k) {
      if (!open_conv::live(px[k], n)) continue;
      const float* q = img + px[k].at;
      float z = 0.f;
#pragma unroll
      for (int j = 0; j < 9; ++j) z = fma(w[j], q[j / 3 * PW + j % 3], z);
      a = fma(dact_f<float, ACT>(z) * lam[k], q[toff], a);
    }
    acc += (double)a;
    if (B - e0 <= IM) break;
  }
  const double v = block_sum<GNT>(acc, sh);
  if (t == 0) dL[co * 9 + tap] = (float)v;
}

template <typename T>
__global__ __launch_bounds__(NT) void k_sgd(size_t n, T lr, const T* g, T* x) {
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT)
    x[i] = x[i] - lr * g[i];
}

template <typename T, typename F>
hipError_t with_act(int act, F&& f) {
  switch (act) {
    case ACT_TANH: return f(std::integral_constant<int, ACT_TANH>{});
    case ACT_RELU: return f(std::integral_constant<int, ACT_RELU>{});
    case ACT_SMOOTHRELU: return f(std::integral_constant<int, ACT_SMOOTHRELU>{});
    case ACT_IDENTITY: return f(std::integral_constant<int, ACT_IDENTITY>{});
  }
  return hipErrorNotSupported;
}

template <typename T>
hipError_t open_fwd_t(const Shape& s, int opening, int nf, int B, const void* y, const void* L, void* u0,
                      hipStream_t st) {
  const int q = s.C * s.H * s.W;
  if (opening == 0) {
    const size_t bytes = (size_t)B * q * sizeof(T);
    if (bytes % 16 || (uintptr_t)u0 % 16 || (uintptr_t)y % 16)
      return hipMemcpyAsync(u0, y, bytes, hipMemcpyDeviceToDevice, st);
    k_copy16<<<grid_for(bytes / 16), NT, 0, st>>>(static_cast<uint4*>(u0), static_cast<const uint4*>(y), bytes / 16);
    return hipGetLastError();
  }
  return with_act<T>(s.act, [&](auto ac) -> hipError_t {
    constexpr int ACT = decltype(ac)::value;
    if (opening == 1)
      k_open_dense<T, ACT><<<dim3((B + OE - 1) / OE, (q + OR - 1) / OR), NT, 0, st>>>((const T*)y, (const T*)L,
                                                                                      (T*)u0, B, q, nf);
    else
      k_open_conv<T, ACT><<<grid_for((size_t)B * q), NT, 0, st>>>((const T*)y, (const T*)L, (T*)u0, B, s.C,
                                                                  s.H, s.W);
    return hipGetLastError();
  });
}

template <typename T>
hipError_t open_grad_t(const Shape& s, int opening, int nf, int B, const void* y, const void* L,
                       const void* lam0, void* dL, hipStream_t st) {
  const int q = s.C * s.H * s.W;
  return with_act<T>(s.act, [&](auto ac) -> hipError_t {
    constexpr int ACT = decltype(ac)::value;
    if (opening == 1) {
      open_grad_dense<T, ACT>((const T*)y, (const T*)L, (const T*)lam0, (T*)dL, B, q, nf, st);
    } else if constexpr (sizeof(T) == 4) {
      if (open_conv::group(s.H, s.W).IM < 1) return hipErrorNotSupported;
      k_open_grad_conv<ACT><<<s.C * 9, GNT, 0, st>>>((const float*)y, (const float*)L, (const float*)lam0, (float*)dL,
                                                     B, s.C, s.H, s.W);
    } else {
      return hipErrorNotSupported;
    }
    return hipGetLastError();
  });
}

}  // namespace

hipError_t launch_copy_rows(void* X, size_t slice_bytes, long src_row, long dst_row0, long dst_step,
                            long count, hipStream_t st) {
  if (count <= 0 || slice_bytes == 0) return hipSuccess;
  const size_t units = slice_bytes / 16;
  // about 8192 workgroups: the rows are split into groups when one row's
  // workgroups are fewer
  const unsigned gx = grid_for(units);
  const long want = std::max<long>(1, std::min<long>(count, (8192 + gx - 1) / gx));
  const long rows = (count + want - 1) / want, groups = (count + rows - 1) / rows;
  if (groups > 65535) return hipErrorInvalidValue;  // the grid's y dimension
  k_copy_rows<<<dim3(gx, (unsigned)groups), NT, 0, st>>>(static_cast<uint4*>(X), units, src_row, dst_row0,
                                                         dst_step, count, rows);
  return hipGetLastError();
}

hipError_t launch_norm_reduce(const double* partial, int n, double* out, hipStream_t st) {
  k_norm_reduce<<<1, NTR, 0, st>>>(partial, n, out);
  return hipGetLastError();
}

hipError_t read_nonfinite(uint32_t* flag, bool clear, hipStream_t st) {
  hipError_t e = hipMemcpyFromSymbolAsync(flag, HIP_SYMBOL(g_nonfinite), sizeof(uint32_t), 0,
                                          hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(st);
  if (e != hipSuccess || !clear || *flag == 0u) return e;
  const uint32_t zero = 0u;
  e = hipMemcpyToSymbolAsync(HIP_SYMBOL(g_nonfinite), &zero, sizeof(uint32_t), 0, hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return e;
  return hipStreamSynchronize(st);
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  k_zero<<<grid_for(bytes / 4), NT, 0, st>>>(static_cast<uint32_t*>(p), bytes / 4);
  return hipGetLastError();
}

hipError_t launch_open_forward(const Shape& s, int opening, int nf, int B, const void* y, const void* L,
                               void* u0, hipStream_t st) {
  return s.dtype == 0 ? open_fwd_t<float>(s, opening, nf, B, y, L, u0, st)
                      : open_fwd_t<double>(s, opening, nf, B, y, L, u0, st);
}

hipError_t launch_open_grad(const Shape& s, int opening, int nf, int B, const void* y, const void* L,
                            const void* lam0, void* dL, hipStream_t st) {
  return s.dtype == 0 ? open_grad_t<float>(s, opening, nf, B, y, L, lam0, dL, st)
                      : open_grad_t<double>(s, opening, nf, B, y, L, lam0, dL, st);
}

// y <- a x + b y (b == 0: y <- a x, whatever y held)
template <typename T>
__global__ __launch_bounds__(NT) void k_axpby(size_t n, double a, const T* x, double b, T* y) {
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT)
    y[i] = b == 0.0 ? (T)(a * (double)x[i]) : (T)(a * (double)x[i] + b * (double)y[i]);
}

// Dot product in fp64 and in a fixed order. Up to DOT_ONE elements one workgroup
// sums in one launch (element t + k NTR per thread, then the threads in a fixed
// tree). Above, workgroup w sums the elements w NT + t (+ k DOT_BLOCKS NT) per thread,
// then its threads in a fixed tree; the second pass adds the DOT_BLOCKS partials in
// the same tree (5.8 us when one thread added them in order, longer than the first
// pass). Two-loop recursion over five arrays, three of them below DOT_ONE: 1701 us
// before, 1596 us now.
constexpr size_t DOT_ONE = 8 * NTR;

template <typename T>
__global__ __launch_bounds__(NTR) void k_dot_one(int n, const T* x, const T* y, double* out) {
  __shared__ double sh[NTR];
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < (int)(DOT_ONE / NTR); ++k) {
    const int i = threadIdx.x + k * NTR;
    if (i < n) s += (double)x[i] * (double)y[i];
  }
  s = block_sum<NTR>(s, sh);
  if (threadIdx.x == 0) out[0] = s;
}

template <typename T>
__global__ __launch_bounds__(NT) void k_dot_part(size_t n, const T* x, const T* y, double* part) {
  __shared__ double sh[NT];
  double s = 0.0;
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)DOT_BLOCKS * NT)
    s += (double)x[i] * (double)y[i];
  s = block_sum<NT>(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ __launch_bounds__(DOT_BLOCKS) void k_dot_final(const double* part, double* out) {
  __shared__ double sh[DOT_BLOCKS];
  const double s = block_sum<DOT_BLOCKS>(part[threadIdx.x], sh);
  if (threadIdx.x == 0) out[0] = s;
}

hipError_t launch_axpby(int dtype, size_t n, double a, const void* x, double b, void* y, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (dtype == 0) k_axpby<float><<<grid_for(n), NT, 0, st>>>(n, a, (const float*)x, b, (float*)y);
  else k_axpby<double><<<grid_for(n), NT, 0, st>>>(n, a, (const double*)x, b, (double*)y);
  return hipGetLastError();
}

template <typename T>
void dot_t(size_t n, const T* x, const T* y, double* out, hipStream_t st) {
  if (n <= DOT_ONE) {
    k_dot_one<T><<<1, NTR, 0, st>>>((int)n, x, y, out);
    return;
  }
  k_dot_part<T><<<DOT_BLOCKS, NT, 0, st>>>(n, x, y, out + 1);
  k_dot_final<<<1, DOT_BLOCKS, 0, st>>>(out + 1, out);
}

hipError_t launch_dot(int dtype, size_t n, const void* x, const void* y, double* out, hipStream_t st) {
  if (dtype == 0) dot_t(n, (const float*)x, (const float*)y, out, st);
  else dot_t(n, (const double*)x, (const double*)y, out, st);
  return hipGetLastError();
}

hipError_t launch_sgd(int dtype, size_t n, double lr, const void* g, void* x, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (dtype == 0) k_sgd<float><<<grid_for(n), NT, 0, st>>>(n, (float)lr, (const float*)g, (float*)x);
  else k_sgd<double><<<grid_for(n), NT, 0, st>>>(n, lr, (const double*)g, (double*)x);
  return hipGetLastError();
}

}  // namespace lp
