// The re-rank kernel for (pair, lambda) codes of more than 32 sub-parts.
#include "rerank_kernel.hpp"

namespace pqt {
PQT_RERANK_VARIANT_DEFINE(pair_long, kPairLong, false)
}  // namespace pqt
