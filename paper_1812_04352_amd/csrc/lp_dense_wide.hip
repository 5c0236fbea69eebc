// Dense fp32 residual layers of width 220 (the hyperspectral network of
// Section 5.1, whose width is the number of spectral bands) on the matrix cores.
//
// At this width a layer step is a real dense contraction (2 q^2 = 96.8 kflop per
// example against 2 q e = 1.8 kB of state traffic), so the kernels are bound by
// the matrix cores, not by HBM, and run their products as split bf16 ones
// (lp_split.h).
//
// A workgroup runs T tiles of 16 examples on NP = 7 waves; the width is padded to
// QP = 224 = 7 panels of 32 features and wave w owns the features of panel w: their
// rows of K_n (or of K_n^T) are the wave's alone, so the weights go from L2 straight
// to its registers, and their state values of all T tiles lie in its registers in
// accumulator layout: register r of block m (0, 1) of tile t in lane l holds feature
// 32 w + 16 m + 4 (l/16) + r of example l%16. What the other waves need of it is the
// B operand, and that is the same layout again: for contraction panel p the eight
// values of a lane are blocks 0 and 1 of wave p. So after each step a wave splits
// its new values and writes them to LDS as fragments [tile][panel][part][lane] of 16
// bytes, one conflict-free write and, for the readers, one conflict-free read per
// lane, with a barrier before and after. A fragment read feeds 12 matrix
// instructions, a weight fragment 6 T; the waves run a whole layer between barriers.
// Padding features (220..223) are never loaded or stored. The weights of a padded
// contraction index are those of a valid one (fetch_a) and meet padded state values of
// zero; the results of a padded row are discarded: the padded values of every new state
// are reset to zero after the activation (sigma(0) is not zero for the smoothed ReLU).
//
// T = 6 takes 126 kB of LDS, one workgroup per CU, two waves per SIMD on three SIMDs
// and one on the fourth; sweeps with fewer workgroups than CUs take T = 4 or 2.
// Streaming K_n through LDS instead, in panels that all waves read for their own 16
// examples, needs a barrier per panel and as much LDS time as matrix time. Finest
// sweeps of 1000 examples and 1024 layers, us: forward FC 1106 (panels, fp32
// instructions), 840 (panels, split products), 725 (this form); forward FRES 1133,
// 890, 780; adjoint FC 1097, 835, 815; adjoint FRES 1433, 1480, 1020. The matrix
// pipes are busy 31 to 36 % of the time in these: a layer's activations, splits and
// barriers come at the same time for all waves, and one workgroup fills the CU.
// (Reading fragments and splitting weights a pair of tiles ahead was not faster: its
// registers spill.)
//
// Sweep modes, the record of sigma' and the FAS bookkeeping follow Algorithm 1
// (Section 3.1) exactly as the other dense kernels do.
#include <stdlib.h>
#include <string.h>

#include "lp_device.h"
#include "lp_internal.h"
#include "lp_split.h"

namespace lp {
namespace wide {

typedef float f32x4 __attribute__((ext_vector_type(4)));
// four floats in global memory, with their element's alignment (the caller's arrays may
// be views into a flat vector)
typedef float f32x4g __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int MODE_SERIAL = 3;

template <int Q>
struct Geo {
  static_assert(Q % 4 == 0, "rows are read as 16-byte vectors");
  static constexpr int QP = (Q + 31) / 32 * 32;  // padded width
  static constexpr int NP = QP / 32;             // panels, waves per workgroup
  static constexpr int NT = 64 * NP;
  static constexpr int NF = 3 * 64 * NP;         // fragments per tile
};

// The lane's place: its panel (wave), lane group and example, and whether its second
// block is real (the first always is: only the last panel is cut short).
template <int Q, int T>
struct Ctx {
  int lane, g, w;
  bool ok1;
  size_t row[T];  // element offset of (example of tile t, feature 32 w + 4 g) in a state row block
  bool on[T];
  __device__ Ctx(int tile, int B) {
    lane = threadIdx.x & 63;
    g = lane >> 4;
    w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    ok1 = 32 * w + 16 + 4 * g < Q;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int e = (tile * T + t) * 16 + (lane & 15);
      on[t] = e < B;
      row[t] = (size_t)(on[t] ? e : 0) * Q + 32 * w + 4 * g;
    }
  }
};

// ------------------------------------------------------------------ rows
template <int T>
using Val = f32x4[T][2];  // a wave's values of its T tiles

// one tile's two blocks at p (the lane's element of the example's row)
__device__ __forceinline__ void load2(f32x4 (&v)[2], const float* __restrict__ p, bool ok1) {
  v[0] = *reinterpret_cast<const f32x4g*>(p);
  v[1] = ok1 ? (f32x4)*reinterpret_cast<const f32x4g*>(p + 16) : f32x4{};
}
__device__ __forceinline__ void store2(float* __restrict__ p, const f32x4 (&v)[2], bool ok1) {
  *reinterpret_cast<f32x4g*>(p) = v[0];
  if (ok1) *reinterpret_cast<f32x4g*>(p + 16) = v[1];
}

// all tiles, from the row block at base; lanes past the batch read example 0's row
// (valid memory; every example is its own column of the products) and store nothing
template <int Q, int T>
__device__ __forceinline__ void load_rows(Val<T>& v, const float* __restrict__ base, const Ctx<Q, T>& c) {
#pragma unroll
  for (int t = 0; t < T; ++t) load2(v[t], base + c.row[t], c.ok1);
}
template <int Q, int T>
__device__ __forceinline__ void store_rows(float* __restrict__ base, const Val<T>& v, const Ctx<Q, T>& c) {
#pragma unroll
  for (int t = 0; t < T; ++t)
    if (c.on[t]) store2(base + c.row[t], v[t], c.ok1);
}

// The sigma' record at element offset off: one byte (0/1) per value for ReLU, fp32
// otherwise.
__device__ __forceinline__ void load_dsig(f32x4 (&d)[2], const void* rec, size_t off, int act, bool ok1) {
  if (act == ACT_RELU) {
    const uint8_t* p = static_cast<const uint8_t*>(rec) + off;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const uint32_t x = m == 0 || ok1 ? *reinterpret_cast<const uint32_t*>(p + 16 * m) : 0u;
#pragma unroll
      for (int r = 0; r < 4; ++r) d[m][r] = (x >> (8 * r)) & 0xffu ? 1.f : 0.f;
    }
  } else {
    load2(d, static_cast<const float*>(rec) + off, ok1);
  }
}
__device__ __forceinline__ void store_dsig(void* rec, size_t off, int act, const f32x4 (&d)[2], bool ok1) {
  if (act == ACT_RELU) {
    uint8_t* p = static_cast<uint8_t*>(rec) + off;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      uint32_t x = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) x |= (d[m][r] != 0.f ? 1u : 0u) << (8 * r);
      if (m == 0 || ok1) *reinterpret_cast<uint32_t*>(p + 16 * m) = x;
    }
  } else {
    store2(static_cast<float*>(rec) + off, d, ok1);
  }
}

// sigma (deriv = false) or sigma' (deriv = true) of every value; padding values are
// reset to zero
template <int ACT, bool DERIV, int T>
__device__ __forceinline__ void apply_one(Val<T>& z) {
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) z[t][m][r] = DERIV ? dact_f<float, ACT>(z[t][m][r]) : act_f<float, ACT>(z[t][m][r]);
}
template <bool DERIV, int T>
__device__ __forceinline__ void apply(Val<T>& z, int act, bool ok1) {
  switch (act) {
    case ACT_TANH: apply_one<ACT_TANH, DERIV, T>(z); break;
    case ACT_RELU: apply_one<ACT_RELU, DERIV, T>(z); break;
    case ACT_SMOOTHRELU: apply_one<ACT_SMOOTHRELU, DERIV, T>(z); break;
    default: if (DERIV) apply_one<ACT_IDENTITY, DERIV, T>(z); break;
  }
#pragma unroll
  for (int t = 0; t < T; ++t)
    if (!ok1) z[t][1] = 0.f;
}

template <int T>
__device__ __forceinline__ void scale(Val<T>& z, float f) {
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int m = 0; m < 2; ++m) z[t][m] *= f;
}

// v = c + (v' - c) (Algorithm 1, the coarse-grid correction of a C-point)
template <int Q, int T>
__device__ __forceinline__ void correct(Val<T>& v, const float* cs, const float* vs, const Ctx<Q, T>& c) {
#pragma unroll
  for (int t = 0; t < T; ++t) {
    f32x4 a[2], b[2];
    load2(a, cs + c.row[t], c.ok1);
    load2(b, vs + c.row[t], c.ok1);
#pragma unroll
    for (int m = 0; m < 2; ++m) v[t][m] = a[m] + (b[m] - a[m]);
  }
}

__device__ __forceinline__ double sq_diff(const f32x4 (&a)[2], const f32x4 (&b)[2]) {
  double acc = 0.0;
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float d = a[m][r] - b[m][r];
      acc += (double)d * (double)d;
    }
  return acc;
}

template <int W>
__device__ __forceinline__ double wg_sum(double v, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < W; ++w) s += red[w];
  return s;
}

// ------------------------------------------------------------------ products
// The wave's weights of one contraction panel on their way to its registers: A
// operand rows 32 w + 16 m + lane % 16, contraction 32 p + 16 h + 4 g + (0..3), of
// K_n (TR false) or of K_n^T. Addresses are a uniform base and 32-bit lane offsets.
// Past the width a valid weight of the same row (or, for a padded row, of row 0) is
// read instead: padded state values are zero, and padded results are discarded.
struct Raw {
  f32x4 r[2][2];
};
template <int Q, bool TR>
__device__ __forceinline__ void fetch_a(Raw& a, const float* __restrict__ Kn, int p, int w, int lane) {
  const int i = lane & 15, k0 = 4 * (lane >> 4);
  const char* base = reinterpret_cast<const char*>(Kn + (TR ? 32 * p * Q : 32 * p));
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const int o = 32 * w + 16 * m + i, oc = o < Q ? o : 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int k = k0 + 16 * h;
      if (32 * (p + 1) > Q) k = 32 * p + k < Q ? k : 0;
      const uint32_t off = 4u * (uint32_t)(TR ? k * Q + oc : oc * Q + k);
      if constexpr (!TR) {
        a.r[m][h] = *reinterpret_cast<const f32x4g*>(base + off);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) a.r[m][h][t] = *reinterpret_cast<const float*>(base + t * 4 * Q + off);
      }
    }
  }
}

// Publishes the wave's values times the sign of the layer that will use them: split,
// panel w of every tile.
template <int Q, int T>
__device__ __forceinline__ void publish(bf16x8* sh, const Val<T>& v, const Ctx<Q, T>& c, float sgn) {
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const Split8 f = split8(sgn * v[t][0], sgn * v[t][1]);
#pragma unroll
    for (int part = 0; part < 3; ++part) sh[((t * Geo<Q>::NP + c.w) * 3 + part) * 64 + c.lane] = f.p[part];
  }
}

constexpr f32x4 ZERO[2] = {f32x4{}, f32x4{}};

// The results that are not finite, again with fp32 instructions (z = init + A v; the
// weights past the width, which a padded state value of zero does not cancel here when
// they are not finite, count as zero).
template <int Q, int T, bool TR>
__device__ __forceinline__ void prod_again(Val<T>& z, const f32x4 (&init)[2], const float* __restrict__ Kn,
                                           const bf16x8* B, const Ctx<Q, T>& c) {
  constexpr int NP = Geo<Q>::NP;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    f32x4 f[2] = {init[0], init[1]};
#pragma unroll 1
    for (int p = 0; p < NP; ++p) {
      Raw q;
      fetch_a<Q, TR>(q, Kn, p, c.w, c.lane);
      Split8 b;
#pragma unroll
      for (int part = 0; part < 3; ++part) b.p[part] = B[((t * NP + p) * 3 + part) * 64];
      const f32x8 x = join8(b);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bool in = 32 * p + 16 * h + 4 * c.g < Q;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int m = 0; m < 2; ++m)
            f[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? q.r[m][h][r] : 0.f, x[4 * h + r], f[m], 0, 0, 0);
      }
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) z[t][m] = pick(z[t][m], f[m]);
  }
}

// z = init + K_n v (or K_n^T v) for the published v (sign included). Two panels of weights are in flight;
// q0, q1 hold panels 0 and 1 on entry and those of the next product (Knext, kind
// NTR; nullptr: none) on return.
template <int Q, int T, bool TR, bool NTR>
__device__ __forceinline__ void prod(Val<T>& z, const f32x4 (&init)[2], const float* __restrict__ Kn, const bf16x8* sh,
                                     const Ctx<Q, T>& c, Raw& q0, Raw& q1, const float* __restrict__ Knext) {
  constexpr int NP = Geo<Q>::NP;
  const bf16x8* B = sh + c.lane;
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int m = 0; m < 2; ++m) z[t][m] = init[m];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    Raw& q = p & 1 ? q1 : q0;
    const Split8 a0 = split8(q.r[0][0], q.r[0][1]), a1 = split8(q.r[1][0], q.r[1][1]);
    if (p + 2 < NP) fetch_a<Q, TR>(q, Kn, p + 2, c.w, c.lane);
#pragma unroll
    for (int t = 0; t < T; t += 2) {
      Split8 b[2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int part = 0; part < 3; ++part) b[u].p[part] = B[(((t + u) * NP + p) * 3 + part) * 64];
      mma_split4(a0, a1, b[0], b[1], z[t][0], z[t][1], z[t + 1][0], z[t + 1][1]);
    }
  }
  if (Knext) {
    fetch_a<Q, NTR>(q0, Knext, 0, c.w, c.lane);
    fetch_a<Q, NTR>(q1, Knext, 1, c.w, c.lane);
  }
  f32x4 sum = z[0][0] + z[0][1];
#pragma unroll
  for (int t = 1; t < T; ++t) sum += z[t][0] + z[t][1];
  if (__builtin_expect(!all_finite(sum), 0)) prod_again<Q, T, TR>(z, init, Kn, B, c);
}

// Work item of linear workgroup id L: the dispatcher deals workgroups to the 8
// XCDs in turn, so item (L % 8) * (n / 8) + L / 8 gives each XCD a contiguous run
// of intervals (all batch tiles of one interval on one XCD: its weights are read
// once into that XCD's L2). Falls back to L when n is not a multiple of 8.
__device__ __forceinline__ void xcd_item(int& tile, int& itv) {
  const unsigned gx = gridDim.x, n = gx * gridDim.y;
  const unsigned L = blockIdx.x + gx * blockIdx.y;
  const unsigned W = n % 8 == 0 ? (L % 8) * (n / 8) + L / 8 : L;
  itv = (int)(W / gx);
  tile = (int)(W - (unsigned)itv * gx);
}

// ------------------------------------------------------------------ forward
template <int Q, int MODE, bool REC, int T>
__global__ __launch_bounds__(Geo<Q>::NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_fwd(SweepArgs a) {
  using G = Geo<Q>;
  __shared__ bf16x8 sh[T * G::NF];
  __shared__ double red[G::NP];
  int tile, k;
  xcd_item(tile, k);
  const int Nc = gridDim.y;
  const Ctx<Q, T> cx(tile, a.B);
  const size_t slice = (size_t)a.B * Q;
  const float* K = static_cast<const float*>(a.K);
  const float* bb = static_cast<const float*>(a.b) + 32 * cx.w + 4 * cx.g;
  float* X = static_cast<float*>(a.X);
  const float* Gr = static_cast<const float*>(a.G);
  const float* Cs = static_cast<const float*>(a.Cs);
  const float* Vn = static_cast<const float*>(a.V);
  const int c = a.c;
  const int nsteps = MODE == MODE_SERIAL ? a.Nl : (MODE == SWEEP_CORRF ? c - 1 : c);
  const float hl = (float)a.hl, hc = (float)a.hc;
  const long kc = MODE == MODE_SERIAL ? 0 : (long)k * c;
  auto layer = [&](long j) { return K + (size_t)(kc + j) * a.stride * (Q * Q); };

  // the final F-relaxation (and a level-0 serial solve) records sigma'(z) of every
  // layer; CORRF then also takes the product of the layer before the next C-point
  constexpr bool rec = REC && (MODE == SWEEP_CORRF || MODE == MODE_SERIAL);
  constexpr bool extra = MODE == SWEEP_CORRF && rec;
  Raw q0, q1;
  if (nsteps > 0 || extra) {
    fetch_a<Q, false>(q0, layer(0), 0, cx.w, cx.lane);
    fetch_a<Q, false>(q1, layer(0), 1, cx.w, cx.lane);
  }
  Val<T> v;
  if (MODE == SWEEP_FC || MODE == MODE_SERIAL) {
    // a pending coarse-grid correction of the previous cycle is applied on the fly
    if (MODE == SWEEP_FC && Vn) correct<Q, T>(v, Cs + (size_t)k * a.cs_stride * slice, Vn + (size_t)k * slice, cx);
    else load_rows<Q, T>(v, X + kc * slice, cx);
    if (MODE == SWEEP_FC && k == 0) store_rows<Q, T>(static_cast<float*>(a.S), v, cx);
  } else if (MODE == SWEEP_FRES) {
    load_rows<Q, T>(v, Cs + (size_t)k * a.cs_stride * slice, cx);
  } else {
    correct<Q, T>(v, Cs + (size_t)k * a.cs_stride * slice, Vn + (size_t)k * slice, cx);
    if (k > 0) store_rows<Q, T>(X + kc * slice, v, cx);
  }
  auto sign = [&](int j) { return layer_sign((size_t)(kc + j) * a.stride); };
  publish<Q, T>(sh, v, cx, sign(0));
  __syncthreads();
  // FRES parks the coarse step's value v + h_c sigma(z) of the first layer in its
  // Gn row and finishes g_{l+1}^{k+1} = v - (that value) after the interval, so it
  // holds no extra registers across the steps
  float* gn = MODE == SWEEP_FRES ? static_cast<float*>(a.Gn) + (size_t)(k + 1) * slice : nullptr;
  auto product = [&](Val<T>& z, int j) {
    const float* bn = bb + (size_t)(kc + j) * a.stride * Q;
    const float sgn = sign(j);
    f32x4 b2[2];
    load2(b2, bn, cx.ok1);
    b2[0] *= sgn;
    b2[1] *= sgn;
    prod<Q, T, false, false>(z, b2, layer(j), sh, cx, q0, q1, j + 1 < nsteps + (extra ? 1 : 0) ? layer(j + 1) : nullptr);
    scale<T>(z, sgn);
  };
  for (int j = 0; j < nsteps; ++j) {
    Val<T> z;
    product(z, j);
    if constexpr (rec) {
      Val<T> dz;
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int m = 0; m < 2; ++m) dz[t][m] = z[t][m];
      apply<true, T>(dz, a.act, cx.ok1);
#pragma unroll
      for (int t = 0; t < T; ++t)
        if (cx.on[t]) store_dsig(a.dsig, (size_t)(kc + j) * a.stride * slice + cx.row[t], a.act, dz[t], cx.ok1);
    }
    apply<false, T>(z, a.act, cx.ok1);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (MODE == SWEEP_FRES && j == 0 && cx.on[t]) {
        const f32x4 cs[2] = {v[t][0] + hc * z[t][0], v[t][1] + hc * z[t][1]};
        store2(gn + cx.row[t], cs, cx.ok1);
      }
#pragma unroll
      for (int m = 0; m < 2; ++m) v[t][m] = v[t][m] + hl * z[t][m];
      if (Gr) {
        f32x4 gv[2];
        load2(gv, Gr + (kc + j + 1) * slice + cx.row[t], cx.ok1);
#pragma unroll
        for (int m = 0; m < 2; ++m) v[t][m] += gv[m];
      }
    }
    if (MODE == SWEEP_CORRF || MODE == MODE_SERIAL) store_rows<Q, T>(X + (kc + j + 1) * slice, v, cx);
    if (j + 1 < nsteps || extra) {
      __syncthreads();  // every read of the old state is done
      publish<Q, T>(sh, v, cx, sign(j + 1));
      __syncthreads();
    }
  }
  if constexpr (extra) {
    // sigma' of the layer before the next C-point, from the last F-point
    Val<T> z;
    product(z, nsteps);
    apply<true, T>(z, a.act, cx.ok1);
#pragma unroll
    for (int t = 0; t < T; ++t)
      if (cx.on[t]) store_dsig(a.dsig, (size_t)(kc + nsteps) * a.stride * slice + cx.row[t], a.act, z[t], cx.ok1);
  }
  if (MODE == SWEEP_FC) {
    store_rows<Q, T>(static_cast<float*>(a.S) + (size_t)(k + 1) * slice, v, cx);
  } else if (MODE == SWEEP_FRES) {
    double acc = 0.0;
    const float* cn = Cs + (size_t)(k + 1) * a.cs_stride * slice;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (!cx.on[t]) continue;
      f32x4 x[2], cs[2];
      load2(x, cn + cx.row[t], cx.ok1);
      load2(cs, gn + cx.row[t], cx.ok1);
      acc += sq_diff(v[t], x);
#pragma unroll
      for (int m = 0; m < 2; ++m) cs[m] = v[t][m] - cs[m];  // g_{l+1}^{k+1}
      store2(gn + cx.row[t], cs, cx.ok1);
      if (a.xn_every > 0 && (k + 1) % a.xn_every == 0)
        store2(static_cast<float*>(a.Xn) + (size_t)(k + 1) * slice + cx.row[t], x, cx.ok1);
      if (k == 0) {
        load2(x, Cs + cx.row[t], cx.ok1);
        store2(static_cast<float*>(a.Xn) + cx.row[t], x, cx.ok1);
      }
    }
    if (a.partial) {
      const double s = wg_sum<G::NP>(acc, red);
      if (threadIdx.x == 0) a.partial[(size_t)k * gridDim.x + tile] = s;
    }
  } else if (MODE == SWEEP_CORRF) {
    if (k == Nc - 1) {
      correct<Q, T>(v, Cs + (size_t)Nc * a.cs_stride * slice, Vn + (size_t)Nc * slice, cx);
      store_rows<Q, T>(X + (size_t)a.Nl * slice, v, cx);
    }
  }
}

// s = sigma'(K_n u^n + b_n) * v of the fine state n, published (times the layer's sign): sigma' from the
// record, or by the forward product (whose weights q0, q1 hold on entry; on return
// they hold the transposed product's). Holds barriers; the caller's reads of sh are
// done.
template <int Q, bool REC, int T>
__device__ __forceinline__ void publish_s(const Val<T>& v, const SweepArgs& a, size_t n, size_t slice, bf16x8* sh,
                                          const Ctx<Q, T>& cx, Raw& q0, Raw& q1) {
  const float sgn = layer_sign(n);
  Val<T> d;
  if constexpr (REC) {
#pragma unroll
    for (int t = 0; t < T; ++t) load_dsig(d[t], a.dsig, n * slice + cx.row[t], a.act, cx.ok1);
  } else {
    const float* Kn = static_cast<const float*>(a.K) + n * (Q * Q);
    load_rows<Q, T>(d, static_cast<const float*>(a.Uf) + n * slice, cx);
    publish<Q, T>(sh, d, cx, sgn);
    __syncthreads();
    f32x4 b2[2];
    load2(b2, static_cast<const float*>(a.b) + n * Q + 32 * cx.w + 4 * cx.g, cx.ok1);
    b2[0] *= sgn;
    b2[1] *= sgn;
    prod<Q, T, false, true>(d, b2, Kn, sh, cx, q0, q1, Kn);
    scale<T>(d, sgn);
    apply<true, T>(d, a.act, cx.ok1);
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int m = 0; m < 2; ++m) d[t][m] = d[t][m] * v[t][m];
  publish<Q, T>(sh, d, cx, sgn);
  __syncthreads();
}

// ------------------------------------------------------------------ adjoint
// Interval k runs from its upper C-point (k+1)c down to kc; step j produces level
// point i = (k+1)c-1-j, linearised at the fine state of index i*stride.
template <int Q, int MODE, bool REC, int T>
__global__ __launch_bounds__(Geo<Q>::NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_adj(SweepArgs a) {
  using G = Geo<Q>;
  __shared__ bf16x8 sh[T * G::NF];
  __shared__ double red[G::NP];
  int tile, k;
  xcd_item(tile, k);
  const int Nc = gridDim.y;
  const Ctx<Q, T> cx(tile, a.B);
  const size_t slice = (size_t)a.B * Q;
  const float* K = static_cast<const float*>(a.K);
  float* X = static_cast<float*>(a.X);
  const float* Gr = static_cast<const float*>(a.G);
  const float* Cs = static_cast<const float*>(a.Cs);
  const float* Vn = static_cast<const float*>(a.V);
  const int c = a.c;
  const int nsteps = MODE == MODE_SERIAL ? a.Nl : (MODE == SWEEP_CORRF ? c - 1 : c);
  const float hl = (float)a.hl, hc = (float)a.hc;
  const long top = MODE == MODE_SERIAL ? (long)a.Nl : (long)(k + 1) * c;
  auto layer = [&](long j) { return K + (size_t)(top - 1 - j) * a.stride * (Q * Q); };

  Raw q0, q1;
  if (nsteps > 0) {
    fetch_a<Q, REC>(q0, layer(0), 0, cx.w, cx.lane);
    fetch_a<Q, REC>(q1, layer(0), 1, cx.w, cx.lane);
  }
  Val<T> v;
  if (MODE == SWEEP_FC || MODE == MODE_SERIAL) {
    if (MODE == SWEEP_FC && Vn)
      correct<Q, T>(v, Cs + (size_t)(k + 1) * a.cs_stride * slice, Vn + (size_t)(k + 1) * slice, cx);
    else load_rows<Q, T>(v, X + top * slice, cx);
    if (MODE == SWEEP_FC && k == Nc - 1) store_rows<Q, T>(static_cast<float*>(a.S) + (size_t)Nc * slice, v, cx);
  } else if (MODE == SWEEP_FRES) {
    load_rows<Q, T>(v, Cs + (size_t)(k + 1) * a.cs_stride * slice, cx);
  } else {
    correct<Q, T>(v, Cs + (size_t)(k + 1) * a.cs_stride * slice, Vn + (size_t)(k + 1) * slice, cx);
    if (k + 1 < Nc) store_rows<Q, T>(X + top * slice, v, cx);
  }
  for (int j = 0; j < nsteps; ++j) {
    const long i = top - 1 - j;
    const size_t n = (size_t)i * a.stride;
    publish_s<Q, REC, T>(v, a, n, slice, sh, cx, q0, q1);
    Val<T> w;
    // the next product: the next step's first one, or the coarse step's with the same weights
    const float* next = j + 1 < nsteps ? layer(j + 1) : MODE == SWEEP_FRES ? layer(j) : nullptr;
    prod<Q, T, true, REC>(w, ZERO, layer(j), sh, cx, q0, q1, next);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (!cx.ok1) w[t][1] = 0.f;
#pragma unroll
      for (int m = 0; m < 2; ++m) v[t][m] = v[t][m] + (layer_sign(n) * hl) * w[t][m];
      if (Gr) {
        f32x4 gv[2];
        load2(gv, Gr + (size_t)i * slice + cx.row[t], cx.ok1);
#pragma unroll
        for (int m = 0; m < 2; ++m) v[t][m] += gv[m];
      }
    }
    if (MODE == SWEEP_CORRF || MODE == MODE_SERIAL) store_rows<Q, T>(X + (size_t)i * slice, v, cx);
    __syncthreads();  // every read of s is done
  }
  double acc = 0.0;  // FRES: squared residual of the lower C-point
  if constexpr (MODE == SWEEP_FRES) {
    // coarse adjoint step from the upper C-point, linearised at the fine state of
    // the interval's last step (sigma' is taken again: same operands, same
    // result), then the residual and the FAS restriction with v the relaxed
    // lower C-point. The step is evaluated exactly as the coarse level evaluates
    // its own steps (c + h_c K_n^T (sigma' * c), the product accumulated from
    // zero), so the FAS right-hand side matches the coarse operator bit for bit;
    // accumulating the product onto c instead rounds every partial sum at the
    // size of c and leaves the iteration a residual floor two orders higher.
    // The residual of the lower C-point is taken first and v is parked in its Gn
    // row, so the state's registers are free during the coarse product.
    const size_t n = (size_t)(top - nsteps) * a.stride;
    float* gn = static_cast<float*>(a.Gn) + (size_t)k * slice;
    const float* cup = Cs + (size_t)(k + 1) * a.cs_stride * slice;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (!cx.on[t]) continue;
      f32x4 x[2];
      load2(x, Cs + (size_t)k * a.cs_stride * slice + cx.row[t], cx.ok1);
      acc += sq_diff(v[t], x);
      if (a.xn_every > 0 && k % a.xn_every == 0)
        store2(static_cast<float*>(a.Xn) + (size_t)k * slice + cx.row[t], x, cx.ok1);
      if (k == Nc - 1) {
        load2(x, Cs + (size_t)Nc * a.cs_stride * slice + cx.row[t], cx.ok1);
        store2(static_cast<float*>(a.Xn) + (size_t)Nc * slice + cx.row[t], x, cx.ok1);
      }
      store2(gn + cx.row[t], v[t], cx.ok1);
    }
    load_rows<Q, T>(v, cup, cx);
    publish_s<Q, REC, T>(v, a, n, slice, sh, cx, q0, q1);
    Val<T> w;
    prod<Q, T, true, true>(w, ZERO, K + n * (Q * Q), sh, cx, q0, q1, nullptr);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (!cx.on[t]) continue;
      f32x4 x[2];
      load2(x, gn + cx.row[t], cx.ok1);
#pragma unroll
      for (int m = 0; m < 2; ++m) x[m] = x[m] - (v[t][m] + (layer_sign(n) * hc) * w[t][m]);  // g_{l+1}^k
      store2(gn + cx.row[t], x, cx.ok1);
    }
  }

  if (MODE == SWEEP_FC) {
    store_rows<Q, T>(static_cast<float*>(a.S) + (size_t)k * slice, v, cx);
  } else if (MODE == SWEEP_FRES) {
    if (a.partial) {
      const double s = wg_sum<G::NP>(acc, red);
      if (threadIdx.x == 0) a.partial[(size_t)k * gridDim.x + tile] = s;
    }
  } else if (MODE == SWEEP_CORRF) {
    if (k == 0) {
      correct<Q, T>(v, Cs, Vn, cx);
      store_rows<Q, T>(X, v, cx);
    }
  }
}

// ------------------------------------------------------------------ residual
// Workgroup (layer n, batch tile): the state residual Phi_n(u^n) - u^{n+1} or the
// adjoint residual lam^{n+1} + h K_n^T (sigma'(K_n u^n + b_n) * lam^{n+1}) - lam^n,
// squared and summed in fp64.
template <int Q, int DIR, int T>
__global__ __launch_bounds__(Geo<Q>::NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_resid(ResidArgs a) {
  using G = Geo<Q>;
  __shared__ bf16x8 sh[T * G::NF];
  __shared__ double red[G::NP];
  const int n = blockIdx.x;
  const Ctx<Q, T> cx(blockIdx.y, a.B);
  const size_t slice = (size_t)a.B * Q;
  const float* U = static_cast<const float*>(a.U);
  const float* L = static_cast<const float*>(a.Lam);
  const float* Kn = static_cast<const float*>(a.K) + (size_t)n * (Q * Q);
  const float h = (float)a.h;
  Raw q0, q1;
  fetch_a<Q, false>(q0, Kn, 0, cx.w, cx.lane);
  fetch_a<Q, false>(q1, Kn, 1, cx.w, cx.lane);
  Val<T> v, z;
  load_rows<Q, T>(v, U + (size_t)n * slice, cx);
  const float sgn = layer_sign(n);
  publish<Q, T>(sh, v, cx, sgn);
  __syncthreads();
  f32x4 b2[2];
  load2(b2, static_cast<const float*>(a.b) + (size_t)n * Q + 32 * cx.w + 4 * cx.g, cx.ok1);
  b2[0] *= sgn;
  b2[1] *= sgn;
  prod<Q, T, false, true>(z, b2, Kn, sh, cx, q0, q1, DIR == DIR_ADJ ? Kn : nullptr);
  scale<T>(z, sgn);
  const float* next = DIR == DIR_FWD ? U + (size_t)(n + 1) * slice : L + (size_t)n * slice;
  if constexpr (DIR == DIR_FWD) {
    apply<false, T>(z, a.act, cx.ok1);
  } else {
    apply<true, T>(z, a.act, cx.ok1);
    load_rows<Q, T>(v, L + (size_t)(n + 1) * slice, cx);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int m = 0; m < 2; ++m) z[t][m] = z[t][m] * v[t][m];
    __syncthreads();
    publish<Q, T>(sh, z, cx, sgn);
    __syncthreads();
    prod<Q, T, true, true>(z, ZERO, Kn, sh, cx, q0, q1, nullptr);
#pragma unroll
    for (int t = 0; t < T; ++t)
      if (!cx.ok1) z[t][1] = 0.f;
    scale<T>(z, sgn);
  }
  double acc = 0.0;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    if (!cx.on[t]) continue;
    f32x4 x[2], f[2];
    load2(x, next + cx.row[t], cx.ok1);
#pragma unroll
    for (int m = 0; m < 2; ++m) f[m] = v[t][m] + h * z[t][m];
    acc += sq_diff(f, x);
  }
  const double s = wg_sum<G::NP>(acc, red);
  if (threadIdx.x == 0) a.partial[(size_t)blockIdx.x * gridDim.y + blockIdx.y] = s;
}

// ------------------------------------------------------------------ gradient
// Workgroup (layer n, batch chunk), GT tiles (64 examples) at a time: the waves form
// s = sigma'(z) * lam^{n+1} (sigma' from the record, or from the forward product),
// then s and u pass through LDS as [example][feature] tiles, 32 examples at a time,
// and dK[i][j] += sum_e s[e][i] u[e][j] runs on v_mfma_f32_32x32x2_f32 with the
// examples as the contraction index (k-slice t pairs examples 2t and 2t+1). The 7 x 7
// output blocks of 32 x 32 are dealt to the seven waves, a row of blocks each, so no
// cross-wave reduction is needed; db sums the s tile's columns. A second pass sums
// the chunk partials in order and scales by h.
constexpr int GT = 4;
template <int Q, bool REC>
__global__ __launch_bounds__(Geo<Q>::NT) void k_grad(GradArgs a) {
  using G = Geo<Q>;
  constexpr int NP = G::NP, TL = G::QP;  // tile pitch: rows 2t and 2t+1 on disjoint banks (QP = 32 mod 64)
  __shared__ __attribute__((aligned(16))) float tiles[2][32 * TL];
  __shared__ bf16x8 sh[REC ? 1 : GT * G::NF];
  const int lane = threadIdx.x & 63, hh = lane >> 5, li = lane & 31;
  const int n = blockIdx.x, chunk = blockIdx.y;
  const int per = (((a.B + a.nchunks - 1) / a.nchunks) + 64 - 1) / 64 * 64;
  const int e0 = chunk * per, e1 = min(a.B, e0 + per);
  const size_t slice = (size_t)a.B * Q;
  const float* U = static_cast<const float*>(a.U) + (size_t)n * slice;
  const float* L = static_cast<const float*>(a.Lam) + (size_t)(n + 1) * slice;
  const float* Kn = static_cast<const float*>(a.K) + (size_t)n * (Q * Q);
  f32x16 acc[NP];
#pragma unroll
  for (int b = 0; b < NP; ++b) acc[b] = 0.f;
  float dbacc = 0.f;  // thread t < Q: column sum of s
  float* st = tiles[0];
  float* ut = tiles[1];
  for (int base = e0; base < e1; base += 16 * GT) {
    const Ctx<Q, GT> cx(base / (16 * GT), e1);
    Val<GT> u, s;
    load_rows<Q, GT>(u, U, cx);
    if constexpr (REC) {
#pragma unroll
      for (int t = 0; t < GT; ++t) load_dsig(s[t], a.dsig, (size_t)n * slice + cx.row[t], a.act, cx.ok1);
    } else {
      Raw q0, q1;
      fetch_a<Q, false>(q0, Kn, 0, cx.w, cx.lane);
      fetch_a<Q, false>(q1, Kn, 1, cx.w, cx.lane);
      const float sgn = layer_sign(n);
      publish<Q, GT>(sh, u, cx, sgn);
      __syncthreads();
      f32x4 b2[2];
      load2(b2, static_cast<const float*>(a.b) + (size_t)n * Q + 32 * cx.w + 4 * cx.g, cx.ok1);
      b2[0] *= sgn;
      b2[1] *= sgn;
      prod<Q, GT, false, false>(s, b2, Kn, sh, cx, q0, q1, nullptr);
      scale<GT>(s, sgn);
      apply<true, GT>(s, a.act, cx.ok1);
    }
#pragma unroll
    for (int t = 0; t < GT; ++t) {
      f32x4 l[2];
      load2(l, L + cx.row[t], cx.ok1);
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        s[t][m] = cx.on[t] ? s[t][m] * l[m] : f32x4{};
        u[t][m] = cx.on[t] ? u[t][m] : f32x4{};
      }
    }
    // two halves of 32 examples
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const int o = (16 * t + (lane & 15)) * TL + 32 * cx.w + 16 * m + 4 * cx.g;
          *reinterpret_cast<f32x4*>(st + o) = s[2 * half + t][m];
          *reinterpret_cast<f32x4*>(ut + o) = u[2 * half + t][m];
        }
      __syncthreads();
#pragma unroll 4
      for (int t = 0; t < 16; ++t) {
        const float sv = st[(2 * t + hh) * TL + 32 * cx.w + li];
        const float* ur = ut + (2 * t + hh) * TL + li;
#pragma unroll
        for (int b = 0; b < NP; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(sv, ur[32 * b], acc[b], 0, 0, 0);
      }
      if (threadIdx.x < Q)
        for (int t = 0; t < 32; ++t) dbacc += st[t * TL + threadIdx.x];
      __syncthreads();
    }
  }
  float* out = static_cast<float*>(a.partial) + ((size_t)n * a.nchunks + chunk) * (Q * Q + Q);
  const int w = threadIdx.x >> 6;
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    const int j = 32 * b + li;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 32 * w + 8 * (r >> 2) + 4 * hh + (r & 3);
      if (i < Q && j < Q) out[(size_t)i * Q + j] = acc[b][r];
    }
  }
  if (threadIdx.x < Q) out[(size_t)Q * Q + threadIdx.x] = dbacc;
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

// ------------------------------------------------------------------ launchers
template <int Q, int T>
void sweep_t(int dir, const SweepArgs& a, dim3 grid, hipStream_t st) {
  constexpr int NT = Geo<Q>::NT;
  const bool rec = a.dsig != nullptr;
  if (dir == DIR_FWD) {
    // only the final F-relaxation (or a level-0 serial solve) writes the sigma' record
    if (a.mode == SWEEP_FC) launch(k_fwd<Q, SWEEP_FC, false, T>, grid, NT, 0, st, a);
    else if (a.mode == SWEEP_FRES) launch(k_fwd<Q, SWEEP_FRES, false, T>, grid, NT, 0, st, a);
    else if (rec) launch(k_fwd<Q, SWEEP_CORRF, true, T>, grid, NT, 0, st, a);
    else launch(k_fwd<Q, SWEEP_CORRF, false, T>, grid, NT, 0, st, a);
  } else if (rec) {
    if (a.mode == SWEEP_FC) launch(k_adj<Q, SWEEP_FC, true, T>, grid, NT, 0, st, a);
    else if (a.mode == SWEEP_FRES) launch(k_adj<Q, SWEEP_FRES, true, T>, grid, NT, 0, st, a);
    else launch(k_adj<Q, SWEEP_CORRF, true, T>, grid, NT, 0, st, a);
  } else {
    if (a.mode == SWEEP_FC) launch(k_adj<Q, SWEEP_FC, false, T>, grid, NT, 0, st, a);
    else if (a.mode == SWEEP_FRES) launch(k_adj<Q, SWEEP_FRES, false, T>, grid, NT, 0, st, a);
    else launch(k_adj<Q, SWEEP_CORRF, false, T>, grid, NT, 0, st, a);
  }
}

// Six tiles per workgroup amortise a layer's weights best; with fewer workgroups than
// that gives two rounds of the 256 CUs, four or two tiles per workgroup finish sooner.
template <int Q>
hipError_t sweep(int dir, const SweepArgs& a, hipStream_t st, int* partials) {
  const long Nc = a.Nl / a.c;
  if (Nc > 65535) return hipErrorNotSupported;  // intervals index the grid's y dimension
  auto groups = [&](int T) { return (a.B + 16 * T - 1) / (16 * T); };
  const int T = groups(6) * Nc >= 512 ? 6 : groups(4) * Nc >= 256 ? 4 : 2;
  const dim3 grid(groups(T), (unsigned)Nc);
  if (partials) *partials = (int)(grid.x * grid.y);
  if (T == 6) sweep_t<Q, 6>(dir, a, grid, st);
  else if (T == 4) sweep_t<Q, 4>(dir, a, grid, st);
  else sweep_t<Q, 2>(dir, a, grid, st);
  return hipGetLastError();
}

template <int Q>
hipError_t serial(int dir, const SerialArgs& s, hipStream_t st) {
  constexpr int NT = Geo<Q>::NT;
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
  // a layer's 194 kB take a CU about as long to read from L2 as two tiles' products
  const dim3 grid((s.B + 31) / 32, 1);
  if (dir == DIR_FWD) {
    if (s.dsig) launch(k_fwd<Q, MODE_SERIAL, true, 2>, grid, NT, 0, st, a);
    else launch(k_fwd<Q, MODE_SERIAL, false, 2>, grid, NT, 0, st, a);
  } else {
    if (s.dsig) launch(k_adj<Q, MODE_SERIAL, true, 2>, grid, NT, 0, st, a);
    else launch(k_adj<Q, MODE_SERIAL, false, 2>, grid, NT, 0, st, a);
  }
  return hipGetLastError();
}

template <int Q>
hipError_t resid(int dir, const ResidArgs& a, hipStream_t st, int* partials) {
  const dim3 grid((unsigned)a.N, (unsigned)((a.B + 63) / 64));
  if (partials) *partials = (int)(grid.x * grid.y);
  if (dir == DIR_FWD) launch(k_resid<Q, DIR_FWD, 4>, grid, Geo<Q>::NT, 0, st, a);
  else launch(k_resid<Q, DIR_ADJ, 4>, grid, Geo<Q>::NT, 0, st, a);
  return hipGetLastError();
}

template <int Q>
hipError_t grad(const GradArgs& a, hipStream_t st) {
  if (a.dsig) launch(k_grad<Q, true>, dim3(a.N, a.nchunks), Geo<Q>::NT, 0, st, a);
  else launch(k_grad<Q, false>, dim3(a.N, a.nchunks), Geo<Q>::NT, 0, st, a);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  const size_t tot = (size_t)a.N * (Q * Q + Q);
  launch(k_grad_final, (unsigned)((tot + 255) / 256), 256, 0, st, a, Q * Q, Q);
  return hipGetLastError();
}

}  // namespace wide

bool wide_width_supported(int q) { return q == 220; }

hipError_t wide_sweep(int q, int dir, const SweepArgs& a, hipStream_t st, int* partials) {
  if (q == 220) return wide::sweep<220>(dir, a, st, partials);
  return hipErrorNotSupported;
}

hipError_t wide_serial(int q, int dir, const SerialArgs& a, hipStream_t st) {
  if (q == 220) return wide::serial<220>(dir, a, st);
  return hipErrorNotSupported;
}

hipError_t wide_resid(int q, int dir, const ResidArgs& a, hipStream_t st, int* partials) {
  if (q == 220) return wide::resid<220>(dir, a, st, partials);
  return hipErrorNotSupported;
}

hipError_t wide_grad(int q, const GradArgs& a, hipStream_t st) {
  if (q == 220) return wide::grad<220>(a, st);
  return hipErrorNotSupported;
}

}  // namespace lp
