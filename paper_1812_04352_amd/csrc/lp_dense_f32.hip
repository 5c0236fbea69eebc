// Dense vector-ALU kernels, fp32 widths 32 and 64.
#include <type_traits>

#include "lp_dense_impl.h"

namespace lp {
namespace {

template <typename F>
hipError_t dispatch(int q, F&& f) {
  if (q == 32) return f(std::integral_constant<int, 32>{});
  if (q == 64) return f(std::integral_constant<int, 64>{});
  return hipErrorNotSupported;
}

}  // namespace

hipError_t dense_sweep_f32(int q, int dir, const SweepArgs& a, hipStream_t st, int* partials) {
  return dispatch(q, [&](auto w) { return dense::sweep<float, decltype(w)::value>(dir, a, st, partials); });
}
hipError_t dense_serial_f32(int q, int dir, const SerialArgs& a, hipStream_t st) {
  return dispatch(q, [&](auto w) { return dense::serial<float, decltype(w)::value>(dir, a, st); });
}
hipError_t dense_resid_f32(int q, int dir, const ResidArgs& a, hipStream_t st, int* partials) {
  return dispatch(q, [&](auto w) { return dense::resid<float, decltype(w)::value>(dir, a, st, partials); });
}
hipError_t dense_grad_f32(int q, const GradArgs& a, hipStream_t st) {
  return dispatch(q, [&](auto w) { return dense::grad<float, decltype(w)::value>(a, st); });
}

}  // namespace lp
