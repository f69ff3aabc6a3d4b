// The re-rank kernel for (pair, lambda) codes, M = 32.
#include "rerank_kernel.hpp"

namespace pqt {
PQT_RERANK_VARIANT_DEFINE(pair16, -16, false)
}  // namespace pqt
