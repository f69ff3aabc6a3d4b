// Host side of the re-rank stage (Sec. 3.2 "vector proposal", Sec. 3.3 "Online computation" Eq. 8-9, Sec. 4
// last kernel): LDS layout, workgroup shape, and the dispatch to the kernel variant for the index's code
// width.  The kernel itself is in rerank_kernel.hpp, compiled per code width in rerank_table*.hip and
// rerank_pair*.hip.
#include <algorithm>

#include "pqt_device.hpp"
#include "rank_head_device.hpp"
#include "rerank_variants.hpp"
#include "traverse_one.hpp"

namespace pqt {

// pair_bytes: of a centroid pair in the table of (pair, lambda) codes, pair_entries: pairs a sub-part has room for
static RerankLds rerank_layout(int M, int k1, int T, int C, int k, int threads, size_t rank_lds, int code_format,
                               int runs_in_lds, size_t pair_bytes, int pair_entries) {
    RerankLds L;
    (void)C;
    L.kpad = next_pow2(k);
    L.scap = 2 * L.kpad < 256 ? 256 : 2 * L.kpad;
    const int want = runs_in_lds < kRunsInLdsMin ? kRunsInLdsMin : runs_in_lds;
    L.rcap = T < want ? T : want;
    size_t o = 0;
    // at offset 0: lookups need no base register.
    // One float per table entry, or (b^2, a^2 - b^2) and c^2 per centroid pair for (pair, lambda) codes.
    L.lut = (uint32_t)o;       o += code_format == 1 ? pair_bytes * (size_t)M * pair_entries : sizeof(float) * M * 256;
    // the survivors are collected when the last score is known: they take the table's place
    L.surv = 0;                o = std::max(o, sizeof(unsigned long long) * (size_t)L.scap);
    L.hist = (uint32_t)o;      o += sizeof(uint32_t) * kHistSize;
    L.part = (uint32_t)o;      o += sizeof(uint32_t) * threads;      // scan scratch of the exact selection
    // everything above is free while a workgroup runs the full bin ranking of its query, which uses
    // the first rank_lds bytes; the arrays below receive its result
    if (o < rank_lds) o = (rank_lds + 15) & ~size_t(15);
    L.a = (uint32_t)o;         o += sizeof(float) * M * k1;
    L.run_src = (uint32_t)o;   o += sizeof(uint32_t) * L.rcap;
    L.run_start = (uint32_t)o; o += sizeof(uint32_t) * (L.rcap + 1);
    L.misc = (uint32_t)o;      o += sizeof(uint32_t) * 16;
    o = (o + 15) & ~size_t(15);
    L.total = (uint32_t)o;
    return L;
}

static RerankLds rerank_layout(int M, int k1, int T, int C, int k, int threads, size_t rank_lds, int code_format,
                               int runs_in_lds) {
    return rerank_layout(M, k1, T, C, k, threads, rank_lds, code_format, runs_in_lds, 3 * sizeof(float), pair_table_stride(k1));
}

size_t rerank_lds_bytes(int M, int k1, int T, int C, int k, int threads, size_t rank_lds, int code_format,
                        int runs_in_lds) {
    return rerank_layout(M, k1, T, C, k, threads, rank_lds, code_format, runs_in_lds).total;
}

// The limit of (pair, lambda) codes is a table of 16 bytes an entry, 128 or 256 of them a sub-part; the table takes less.
size_t rerank_limit_bytes(int M, int k1, int T, int C, int k, int threads, int code_format, int runs_in_lds) {
    return rerank_layout(M, k1, T, C, k, threads, 0, code_format, runs_in_lds, 16, k1 * (k1 - 1) / 2 <= 128 ? 128 : 256).total;
}

void rerank_shape(int C, int M, int code_format, int* threads, int* keys_per_thread) {
    int t = 256;
    while (t < 1024 && C > kKeysPerThread * t) t *= 2;
    (void)M;
    (void)code_format;
    *threads = t;
    *keys_per_thread = kKeysPerThread;
}

// (pair, lambda) codes of any length: four pieces at a time take registers, and with them half of the wavefronts.  10,000 queries, one
// and four pieces, us: M = 24, 4 centroids, 1,831 candidates 202 and 291, 7,324 664 and 933; M = 28 253 and 332, 857 and 1,075; M = 36, 6
// centroids, 813 candidates 228 and 268, 3,255 714 and 638, 6,510 1,221 and 1,065; M = 40, 4 centroids 378 and 376, 1,495 and 1,190.
static bool long_pair_code(int M) { return M > 32; }

int rerank_fused_tuples_per_thread() { return kFusedPer; }

hipError_t launch_rerank(const RerankArgs& a_in, const RankArgs* fused, hipStream_t s) {
    if (a_in.nq <= 0) return hipSuccess;
    RerankArgs a = a_in;
    a.pair_stride = pair_table_stride(a.k1);
    const bool taps = a.n_cand || a.cand_ids || a.scores || a.lut;
    RankArgs rk = {};
    RankOffsets RL = {};
    if (fused) {
        if (taps || fused->P != 2) return hipErrorInvalidValue;
        rk = *fused;
        RL = rank_offsets(rk.P, rk.R, rk.T, rk.hashed, false, rk.t_mid);
        if (RL.Tcap > rerank_fused_tuples_per_thread() * a.threads) return hipErrorInvalidValue;
        // the wavefront's two lists lie at the start of the workgroup's LDS (table, survivor list and
        // histogram are not in use yet, and the arrays that receive the result come after them)
        static_assert(sizeof(HeadLds) <= sizeof(uint32_t) * kHistSize, "the lists must end before the arrays that are live");
        a.mid_T1 = RL.Tcap < kHeadT ? RL.Tcap : kHeadT;
        RL.force = RL.Tmid <= a.mid_T1 ? 1 : 0;       // so many tuples have been tried by then
        a.mid_npairs = head_pair_count(a.mid_T1);
    }
    if (a.keys_per_thread != kKeysPerThread || a.C > a.keys_per_thread * a.threads) return hipErrorInvalidValue;
    if (a.threads % 256 != 0) return hipErrorInvalidValue;             // a thread builds the table entries of one code value
    if (a.code_format == 1 && a.lut) return hipErrorInvalidValue;      // that tap is the one-byte format's table
    const RerankLds L = rerank_layout(a.M, a.k1, a.T, a.C, a.k, a.threads, fused ? RL.total : 0, a.code_format, a.runs_in_lds);
    const bool f = fused != nullptr;
    if (a.code_format == 1) {
        // word-wise variants for the plain entry point; the tapped one takes the kernel for any length.  Codes of six and sixteen words take 128
        // registers, so that one workgroup of 1,024 threads fits a compute unit and two of the kernel for any length do: more queries than compute
        // units in such workgroups go there, those of sixteen words where the kernel ranks as well or with few candidates.  700 and 1,000 queries
        // by words and by pieces, ranking too: M = 12: 1,030 candidates 49 and 68 us, 45 and 61, 2,300 129 and 160, 112 and 131; M = 32: 1,600
        // candidates 66 and 90, 59 and 70, 4,096 100 and 123, 84 and 105, 9,150 200 and 259, 185 and 232; without the ranking, 1,000 and 2,000
        // queries: M = 12: 10,700 candidates 118 and 213, 108 and 187, M = 32: 8,540 165 and 255, 190 and 299.  (Batches of 257 to 1,024 queries
        // come here where they are not answered in one launch.)
        const bool by_bytes = a.threads == 1024 && a.nq > 256 && (a.M == 12 || (a.M == 32 && (f || a.C <= 2048)));
        switch (taps || by_bytes || a.M % 2 ? 0 : a.M / 2) {
            case 2: return launch_rerank_pair2(a, L, rk, RL, taps, f, s);
            case 4: return launch_rerank_pair4(a, L, rk, RL, taps, f, s);
            case 6: return launch_rerank_pair6(a, L, rk, RL, taps, f, s);
            case 8: return launch_rerank_pair8(a, L, rk, RL, taps, f, s);
            case 16: return launch_rerank_pair16(a, L, rk, RL, taps, f, s);
            default:
                if (long_pair_code(a.M) && !taps) return launch_rerank_pair_long(a, L, rk, RL, taps, f, s);
                return launch_rerank_pair_bytes(a, L, rk, RL, taps, f, s);
        }
    }
    switch ((a.M % 4 == 0) ? a.M / 4 : 0) {
        case 1: return launch_rerank_table1(a, L, rk, RL, taps, f, s);
        case 2: return launch_rerank_table2(a, L, rk, RL, taps, f, s);
        case 3: return launch_rerank_table3(a, L, rk, RL, taps, f, s);
        case 4: return launch_rerank_table4(a, L, rk, RL, taps, f, s);
        case 8: return launch_rerank_table8(a, L, rk, RL, taps, f, s);
        default: return launch_rerank_table0(a, L, rk, RL, taps, f, s);
    }
}

// Layout of the kernel for small batches within `room` bytes of LDS: the ranking behind the table, or in its place.  False: it does not
// take these arguments.
static bool small_query_layout(const RerankArgs& a, const RankArgs& rk, const TraverseArgs& tr, size_t room, RankOffsets& RL, RerankLds& L,
                               SmallQuery& sm) {
    if (!traverse_one_possible(tr)) return false;
    RL = rank_offsets(rk.P, rk.R, rk.T, rk.hashed, true, rk.t_mid);
    if (RL.Tcap > 4 * a.threads || a.C > kKeysPerThread * a.threads) return false;
    const size_t ranking = (RL.total + 15) & ~size_t(15);
    for (sm.late_table = 0; sm.late_table < 2; ++sm.late_table) {
        L = rerank_layout(a.M, a.k1, a.T, a.C, a.k, a.threads, sm.late_table ? ranking : 0, a.code_format, a.runs_in_lds);
        size_t o = L.total;
        sm.off_ranking = sm.late_table ? 0u : (uint32_t)o;   o += sm.late_table ? 0 : ranking;
        sm.off_traverse = (uint32_t)o;                       o += traverse_one_layout(tr.D, tr.P, tr.k1, tr.k2, tr.M, tr.w).total;
        sm.off_head = (uint32_t)o;                           o += (sizeof(HeadLds) + 15) & ~size_t(15);
        sm.off_tables = (uint32_t)o;                         o += 2 * kHeadPairs;
        sm.lds = (uint32_t)o;
        if (o <= room) return true;
    }
    return false;
}

bool small_query_fits(const RerankArgs& a, const RankArgs& rk, const TraverseArgs& tr, size_t room) {
    RankOffsets RL;
    RerankLds L;
    SmallQuery sm;
    return small_query_layout(a, rk, tr, room, RL, L, sm);
}

hipError_t launch_small_query(const RerankArgs& a_in, const RankArgs& rk, const TraverseArgs& tr, bool head, const StaticOrder* fixed,
                              size_t room, hipStream_t s) {
    if (a_in.nq <= 0) return hipSuccess;
    RerankArgs a = a_in;
    a.pair_stride = pair_table_stride(a.k1);
    a.early = 0;
    RankOffsets RL;
    RerankLds L;
    SmallQuery sm;
    if (a.keys_per_thread != kKeysPerThread || a.n_cand || a.cand_ids || a.scores || a.lut || !small_query_layout(a, rk, tr, room, RL, L, sm))
        return hipErrorInvalidValue;
    sm.levels = HeadLevels{};
    sm.fixed = fixed ? *fixed : StaticOrder{};
    if (head && !fixed && rk.P == 2)
        for (int l = 0; l < 2; ++l) {
            const int t = 32 << l;
            sm.levels.T1[l] = RL.Tcap < t ? RL.Tcap : t;
            sm.levels.npairs[l] = head_pair_count(sm.levels.T1[l]);
        }
    if (a.code_format == 1) {
        switch (a.M % 2 ? 0 : a.M / 2) {
            case 2: return launch_query_pair2(a, L, rk, RL, tr, sm, s);
            case 4: return launch_query_pair4(a, L, rk, RL, tr, sm, s);
            case 6: return launch_query_pair6(a, L, rk, RL, tr, sm, s);
            case 8: return launch_query_pair8(a, L, rk, RL, tr, sm, s);
            case 16: return launch_query_pair16(a, L, rk, RL, tr, sm, s);
            default:
                if (long_pair_code(a.M)) return launch_query_pair_long(a, L, rk, RL, tr, sm, s);
                return launch_query_pair_bytes(a, L, rk, RL, tr, sm, s);
        }
    }
    switch ((a.M % 4 == 0) ? a.M / 4 : 0) {
        case 1: return launch_query_table1(a, L, rk, RL, tr, sm, s);
        case 2: return launch_query_table2(a, L, rk, RL, tr, sm, s);
        case 3: return launch_query_table3(a, L, rk, RL, tr, sm, s);
        case 4: return launch_query_table4(a, L, rk, RL, tr, sm, s);
        case 8: return launch_query_table8(a, L, rk, RL, tr, sm, s);
        default: return launch_query_table0(a, L, rk, RL, tr, sm, s);
    }
}

hipError_t configure_rerank(size_t max_dynamic_lds) {
    hipError_t (*const all[])(size_t) = {configure_rerank_table0, configure_rerank_table1, configure_rerank_table2,
                                         configure_rerank_table3, configure_rerank_table4, configure_rerank_table8,
                                         configure_rerank_pair_bytes, configure_rerank_pair_long, configure_rerank_pair2, configure_rerank_pair4,
                                         configure_rerank_pair6, configure_rerank_pair8, configure_rerank_pair16};
    for (auto fn : all) {
        const hipError_t e = fn(max_dynamic_lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace pqt
