// The re-rank kernel for one-byte codes, M = 12.
#include "rerank_kernel.hpp"

namespace pqt {
PQT_RERANK_VARIANT_DEFINE(table3, 3, true)
}  // namespace pqt
