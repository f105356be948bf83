// The general kernels in FP32, and the choice of precision.
#include "generic_engine.hpp"

namespace psdns {
Ops ops_general_f64();
Ops ops_general(int precision) { return precision == 32 ? GEngine<float>::ops() : ops_general_f64(); }
// (z, y) lines per block of the x pass
int general_x_lines(int n, int precision, int batch) {
  const gen::Factors f = precision == 32 ? gen::step_factors<float>(n) : gen::step_factors<double>(n);
  return gen::x_shape(f, precision == 32 ? 8 : 16, (long long)n * n * batch).lw;
}
}  // namespace psdns
