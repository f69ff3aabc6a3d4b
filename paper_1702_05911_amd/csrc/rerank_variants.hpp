// The re-rank kernel is compiled once per code width, each width in a translation unit of its own
// (rerank_table*.hip: one byte per sub-part, M = 4, 8, 12, 16, 32 or any; rerank_pair*.hip: (pair, lambda)
// codes, M = 4, 8, 12, 16, 32 word-wise or any in pieces of eight sub-parts; the number in the name counts 32-bit words).  Read byte by
// byte, a candidate cost a load per byte: 3,217 queries x 3,001 candidates of 24 bytes, ranking included, took 456 us, read as words 339
// (and 140 with the ranking in a kernel of its own).  This header declares their launchers.
#pragma once
#include "pqt_kernels.hpp"
#include "rank_head_device.hpp"

namespace pqt {

struct RerankLds {
    int kpad, scap, rcap;
    uint32_t surv, lut, a, run_src, run_start, hist, part, misc, total;
};

// What the kernel that answers a query of a small batch has besides: its LDS, and the tuples the first wavefront ranks by itself
// (T1[0] = 0: none), or the fixed order.
struct SmallQuery {
    HeadLevels levels;
    StaticOrder fixed;               // the fixed bin order (table null: by summed distance)
    uint32_t off_traverse, off_tables, off_ranking, off_head, lds;
    int late_table;                  // the ranking has the table's place: it is built afterwards
};

#define PQT_RERANK_VARIANT_DECLARE(NAME)                                                                               \
    hipError_t launch_rerank_##NAME(const RerankArgs& a, const RerankLds& L, const RankArgs& rk, const RankOffsets& RL, \
                                    bool taps, bool fused, hipStream_t s);                                             \
    hipError_t launch_query_##NAME(const RerankArgs& a, const RerankLds& L, const RankArgs& rk, const RankOffsets& RL,  \
                                   const TraverseArgs& tr, const SmallQuery& sm, hipStream_t s);                       \
    hipError_t configure_rerank_##NAME(size_t max_dynamic_lds);

PQT_RERANK_VARIANT_DECLARE(table0)
PQT_RERANK_VARIANT_DECLARE(table1)
PQT_RERANK_VARIANT_DECLARE(table2)
PQT_RERANK_VARIANT_DECLARE(table3)
PQT_RERANK_VARIANT_DECLARE(table4)
PQT_RERANK_VARIANT_DECLARE(table8)
PQT_RERANK_VARIANT_DECLARE(pair_bytes)
PQT_RERANK_VARIANT_DECLARE(pair_long)
PQT_RERANK_VARIANT_DECLARE(pair2)
PQT_RERANK_VARIANT_DECLARE(pair4)
PQT_RERANK_VARIANT_DECLARE(pair6)
PQT_RERANK_VARIANT_DECLARE(pair8)
PQT_RERANK_VARIANT_DECLARE(pair16)

// compile-time constants the host side needs as well
constexpr int kHistBits = 10;
constexpr int kHistSize = 1 << kHistBits;
constexpr int kFusedPer = 4;         // tuples per thread the in-kernel bin ranking may hold
constexpr int kKeysPerThread = 20;   // candidates a thread scores; C <= kKeysPerThread * workgroup size
constexpr int kRunsInLdsMin = 64;    // at least this many runs of a query are kept in LDS (see RerankArgs::runs_in_lds)

// (pair, lambda) codes: entries per sub-part in the LDS table of centroid pairs (128 while the pairs fit)
inline int pair_table_stride(int k1) { return k1 < 3 ? 2 : (k1 * (k1 - 1) / 2 + 1) & ~1; }

}  // namespace pqt
