// The general kernels in FP64.
#include "generic_engine.hpp"

namespace psdns {
Ops ops_general_f64() { return GEngine<double>::ops(); }
}  // namespace psdns
