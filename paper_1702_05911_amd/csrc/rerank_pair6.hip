// The re-rank kernel for (pair, lambda) codes, M = 12.
#include "rerank_kernel.hpp"

namespace pqt {
PQT_RERANK_VARIANT_DEFINE(pair6, -6, false)
}  // namespace pqt
