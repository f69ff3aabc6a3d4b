// Device code of the re-rank kernel: vector proposal, re-ranking by line quantisation and the final ordering
// (Sec. 3.2 "vector proposal", Sec. 3.3 "Online computation" Eq. 8-9, Sec. 4 last kernel).
//
// One workgroup per query.
//   * the per-query table LUT[m][c] of Eq. 9 summands is built in LDS from the level-1
//     sub-part distances the traversal already produced (no new distance is computed);
//   * codes are stored bin-major beside the ids, so the candidates of a proposed slot are one
//     contiguous run.  A wavefront scores a contiguous piece of the candidate list, 64 positions
//     (one window) after the other, consecutive lanes reading consecutive codes (coalesced),
//     eight windows in flight; where runs are long (eight candidates or more on average) it
//     walks the run list as one, with scalar control and one compare and select per run boundary,
//     where they are short every thread searches the list for its own position.  The id array is
//     only touched for the few survivors;
//   * score = sum over m = 0..M-1, in that order, of LUT[m][code[m]] in fp32;
//   * a thread scores at most twenty candidates and keeps their keys (ordered score bits) in
//     registers through the selection: with eight workgroups per compute unit the vector ALU is
//     busy most of the time on a cache-resident index, so what counts is the number of vector
//     instructions per candidate and how many queries a compute unit has in flight, which is set
//     by the LDS a workgroup holds -- a key array in LDS would double it;
//   * the k best by (score, id): one 1024-bin histogram over the ordered score bits between the
//     smallest and largest score of the query; the first wavefront locates the bin b that holds the
//     k-th smallest; the keys in bins <= b (a superset of the answer, normally a few more
//     than k) are appended to a short list with their positions, their ids fetched, and the
//     (score bits, id) keys sorted in registers.  If the superset does not fit (heavily tied
//     scores) an exact radix select on score bits, then on ids, picks exactly k.
#pragma once
#include <type_traits>

#include "rank_head_device.hpp"
#include "rerank_variants.hpp"
#include "traverse_one.hpp"

namespace pqt {


constexpr int kCountRankMax = 32;    // survivors ordered by counting ranks up to this many, else sorted
constexpr int kWalkMinRun = 8;       // mean run length from which a wavefront walks the run list together
constexpr int kMarkMinRun = 5, kMarkMaxRun = 32;   // and from which to which it marks it (see MarkedRuns)
constexpr int kSurvPer = 8;          // survivors a thread places: those of k = 1024 with 256 threads
constexpr int kRunPrefetch = 64;     // runs fetched before the run count is known

// The run list of one query: the first rcap runs in LDS, any further ones in memory.  The LDS arrays
// are named by their byte addresses (the kernels here have no static LDS, so the dynamic LDS starts
// at address 0; the launcher checks that).
typedef __attribute__((address_space(3))) const uint32_t lds_cuint;
struct RunList {
    uint32_t src, start;       // LDS addresses of run_src / run_start
    const uint2* mem;          // runs of this query in memory
    int rcap, nr;
    uint32_t nc;
    __device__ __forceinline__ uint32_t start_at(int r) const {   // r <= nr
        return r < rcap || r == nr && nr <= rcap ? *reinterpret_cast<lds_cuint*>((uintptr_t)(start + 4u * (uint32_t)r))
                                                 : (r < nr ? mem[r].y : nc);
    }
    __device__ __forceinline__ uint32_t src_at(int r) const {     // r < nr
        return r < rcap ? *reinterpret_cast<lds_cuint*>((uintptr_t)(src + 4u * (uint32_t)r)) : mem[r].x;
    }
};

// Position p of the candidate list -> position in ids/codes: the run r with
// start(r) <= p < start(r+1), found in `steps` = ceil(log2(nr)) halvings.
__device__ __forceinline__ uint32_t source_of(uint32_t p, int steps, const RunList& R) {
    int lo = 0, hi = R.nr;
    for (int s = 0; s < steps; ++s) {
        const int mid = (lo + hi) >> 1;
        const bool ge = R.start_at(mid) <= p;
        lo = ge ? mid : lo;
        hi = ge ? hi : mid;
    }
    return R.src_at(lo) + (p - R.start_at(lo));
}

// One pass of a most-significant-digit radix select (exact fallback).  Counts, among the items whose
// key agrees with `prefix` on the bits of `mask`, the digit (key >> shift) & (2^bits - 1); finds the
// digit holding the item of 1-based rank `need`.  out[0] = digit, out[1] = rank inside it, out[2] =
// size of the chosen digit's bucket.  each_key(f) calls f(key) for every item of the calling thread.
// All threads must call it; ends with a barrier.
template <typename EachKey>
__device__ __forceinline__ void radix_select_pass(uint32_t prefix, uint32_t mask, int shift, int bits, uint32_t need,
                                                  uint32_t* hist, uint32_t* part, uint32_t* out, EachKey each_key) {
    const int tid = threadIdx.x, nt = blockDim.x;
    const int nb = 1 << bits;
    for (int e = tid; e < nb; e += nt) hist[e] = 0;
    __syncthreads();
    each_key([&](uint32_t key) {
        if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & (uint32_t)(nb - 1)], 1u);
    });
    __syncthreads();
    const int chunk = (nb + nt - 1) / nt;
    const int lo = min(tid * chunk, nb), hi = min(lo + chunk, nb);
    uint32_t s = 0;
    for (int e = lo; e < hi; ++e) s += hist[e];
    part[tid] = s;
    __syncthreads();
    for (int off = 1; off < nt; off <<= 1) {
        uint32_t v = (tid >= off) ? part[tid - off] : 0u;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    s = (tid > 0) ? part[tid - 1] : 0u;
    for (int e = lo; e < hi; ++e) {
        const uint32_t c = hist[e];
        if (s < need && need <= s + c) {
            out[0] = (uint32_t)e;
            out[1] = need - s;
            out[2] = c;
        }
        s += c;
    }
    __syncthreads();
}

// misc words
enum { kMin = 0, kMax = 1, kSel = 2, kSelCount = 3, kNumSurv = 4, kFullBin = 5, kRadix = 8, kRanked = 12 };

// LUT[m][c] read through an LDS address formed from the code byte alone: the table sits at LDS
// address 0 (the kernels here have no static LDS; the launcher checks that), so the address is
// c * 4 plus the compile-time offset m * 1024 -- one sub-dword shift per lookup.
typedef __attribute__((address_space(3))) const float lds_cfloat;
__device__ __forceinline__ float lut_at(int m, uint32_t c) {
    return *reinterpret_cast<lds_cfloat*>((uintptr_t)((c << 2) + (uint32_t)m * 1024u));
}
// the same for byte B of a code word: four times the byte in ONE sub-dword shift, for the low byte too
// (for which the compiler would shift the whole word and mask)
template <int B>
__device__ __forceinline__ float lut_at_byte(int m, uint32_t word) {
    uint32_t addr;
    if constexpr (B == 0)
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0"
            : "=v"(addr) : "v"(2u), "v"(word));
    else
        addr = ((word >> (8 * B)) & 0xffu) << 2;
    return *reinterpret_cast<lds_cfloat*>((uintptr_t)(addr + (uint32_t)m * 1024u));
}

// The run a thread's current candidate position lies in, kept in registers: positions of a thread
// only grow, so the run only moves forwards and the run list is read only when a position crosses
// into another run.
struct RunCursor {
    int run;
    uint32_t next_start;   // run_start[run + 1]
    uint32_t delta;        // run_src[run] - run_start[run]: position in ids/codes = candidate position + delta
};

// Where a wavefront stands in the run list while it walks its piece of the candidate list, 64
// positions (one window) at a time.  Lane l holds run blk0 + l of the list; r (the same in every
// lane) is the first run that starts after the windows done so far, dcur the offset
// run_src - run_start of run r - 1.  Everything that steers the walk is wavefront-uniform, so the
// per-position work is one compare and one select per run boundary inside the window.
struct WaveRuns {
    uint32_t v_src, v_start;   // run blk0 + lane (v_start = 0xffffffff past the end of the list)
    int blk0, r;
    uint32_t dcur;
    uint32_t next_s;           // start of run r, 0xffffffff when the list is used up
    __device__ __forceinline__ void load(const RunList& R, int first, int lane) {
        blk0 = first;
        const int idx = first + lane;
        v_start = 0xffffffffu;
        v_src = 0u;
        if (idx < R.nr) {
            v_start = R.start_at(idx);
            v_src = R.src_at(idx);
        }
    }
    __device__ __forceinline__ void fetch_next(const RunList& R, int lane) {
        if (r >= R.nr) {
            next_s = 0xffffffffu;
            return;
        }
        if (r - blk0 >= kWave) load(R, r & ~(kWave - 1), lane);
        next_s = (uint32_t)__builtin_amdgcn_readlane((int)v_start, r - blk0);
    }
    // positions [wbase, ...) come next: r = number of runs that start at or before wbase (at least one)
    __device__ __forceinline__ void seek(const RunList& R, uint32_t wbase, int lane) {
        int b = 0;
        while ((b + 1) * kWave < R.nr &&
               (uint32_t)__builtin_amdgcn_readfirstlane((int)R.start_at((b + 1) * kWave)) <= wbase)
            ++b;
        load(R, b * kWave, lane);
        const int cnt = __popcll(__ballot(v_start <= wbase));
        r = b * kWave + cnt;
        dcur = (uint32_t)__builtin_amdgcn_readlane((int)(v_src - v_start), cnt > 0 ? cnt - 1 : 0);
        fetch_next(R, lane);
    }
    // offset of every lane's position wb + lane (wb: multiple of 64, not below the last window's);
    // a window without a run boundary costs one scalar compare
    __device__ __forceinline__ uint32_t window(const RunList& R, uint32_t wb, int lane) {
        uint32_t delta = dcur;
        while (next_s < wb + kWave) {
            const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)v_src, r - blk0) - next_s;
            delta = wb + (uint32_t)lane >= next_s ? d : delta;
            dcur = d;
            ++r;
            fetch_next(R, lane);
        }
        return delta;
    }
};

// The same walk for runs of medium length, where a window of 64 positions meets several boundaries and each cost the walk above
// half a dozen vector instructions.  Lane l holds run first + l, `first` being the run the group of windows starts in; the
// lanes whose run starts inside the group put their number at that position of a byte array in LDS, and a prefix maximum
// along the positions names every position's run: a dozen instructions per window, whatever the number of boundaries.
// 5,003 queries x 10,000 candidates in runs of ten: the whole call 553 -> 518 us.
struct MarkedRuns {
    uint32_t v_start, v_delta;   // run first + lane: start (0xffffffff past the list), position in ids/codes - candidate position
    int first;
    uint32_t carry;              // run (counted from first) of the last position looked up
    bool many;                   // the group may reach past the 64 runs held: every thread searches the list
    __device__ __forceinline__ void load(const RunList& R, int f, int lane) {
        first = f;
        const int idx = f + lane;
        v_start = 0xffffffffu;
        v_delta = 0u;
        if (idx < R.nr) {
            v_start = R.start_at(idx);
            v_delta = R.src_at(idx) - v_start;
        }
    }
    // the run of position p, not below the last one asked for
    __device__ __forceinline__ void seek(const RunList& R, uint32_t p, int lane) {
        for (;;) {
            const int cnt = __popcll(__ballot(v_start <= p));      // runs held that start at or before p: at least one
            if (cnt == 1) return;
            load(R, first + cnt - 1, lane);
        }
    }
    // positions [p0, p0 + span) come next; marks: this wavefront's bytes, span <= 256
    __device__ __forceinline__ void group(const RunList& R, uint32_t p0, int span, int lane, uint32_t marks) {
        typedef __attribute__((address_space(3))) uint32_t lds_word;
        typedef __attribute__((address_space(3))) uint8_t lds_byte;
        seek(R, p0, lane);
        carry = 0u;
        many = first + kWave < R.nr && (uint32_t)__builtin_amdgcn_readlane((int)v_start, kWave - 1) < p0 + (uint32_t)span;
        wave_lds_order();
        *reinterpret_cast<lds_word*>((uintptr_t)(marks + 4u * (uint32_t)lane)) = 0u;
        wave_lds_order();
        const uint32_t at = v_start - p0;                        // lane 0: not inside (its run starts at or before p0)
        if (lane > 0 && at < (uint32_t)span) *reinterpret_cast<lds_byte*>((uintptr_t)(marks + at)) = (uint8_t)lane;
        wave_lds_order();
    }
    // offset of position p = p0 + 64 * w + lane of the group
    __device__ __forceinline__ uint32_t window(const RunList& R, uint32_t p, bool wanted, int w, int lane, uint32_t marks) {
        typedef __attribute__((address_space(3))) const uint8_t lds_cbyte;
        if (many) {                                              // the same for the wavefront
            uint32_t delta = 0u;
            if (wanted) {
                int lo = first, hi = R.nr;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    const bool ge = R.start_at(mid) <= p;
                    lo = ge ? mid : lo;
                    hi = ge ? hi : mid;
                }
                delta = R.src_at(lo) - R.start_at(lo);
            }
            return delta;
        }
        const uint32_t mark = *reinterpret_cast<lds_cbyte*>((uintptr_t)(marks + (uint32_t)lane + (uint32_t)(w * kWave)));
        const uint32_t run = max(wave_inclusive_max(mark), carry);
        carry = (uint32_t)__builtin_amdgcn_readlane((int)run, kWave - 1);
        return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(run << 2), (int)v_delta);
    }
};

// How a wavefront finds its candidates' places (RUNS of score_batch)
enum { kSearchRuns, kWalkRuns, kMarkRuns };

// (pair, lambda level) codes: the summand of Eq. 9 for one sub-part from the pair's LDS entries, (b^2, a^2 - b^2) of all sub-parts and
// behind them c^2, and the level; lambda = (level - 96) / 16 is exact in fp32.  A read of 8 bytes and one of 4: the pairs of a
// wavefront are as good as random, and one read of 16 (with a fourth word unused) waits for bank conflicts about as long as both
// together, its table twice; a sub-part has as many entries as there are pairs, not the next power of two (3,217 queries x 3,001
// candidates, 190 pairs, M = 12: the kernel 142 -> 88 us; 4 workgroups a compute unit instead of 3).
// MW < 0 selects this code format: kPairLambda and kPairLong any M, else -(words per code).  Any M: a lane reads its candidate's code
// in pieces of eight sub-parts, one at a time, of long codes four.  The cache lines of a lane's code have to last from its first load to its
// last: with a load per sub-part and as many wavefronts as the small tables leave room for they are fetched again and again.  10,000
// queries, 8 centroids, 7,324 candidates, ms, a load per sub-part, a piece, four pieces: M = 56 -, 3.7 and 1.7, M = 64 11.7, 5.6 and 1.7 (of
// two bytes and one workgroup a compute unit, as long as a pair had 16 bytes: 3.2 and 3.5); 16 centroids, M = 24, 1,831 candidates
// 0.52 and 0.47.
constexpr int kPairLambda = -1, kPairLong = -64;
constexpr int code_words(int MW) { return MW > 0 ? MW : (MW == kPairLambda || MW == kPairLong ? 0 : -MW); }     // 0: as many as M says
template <int MW>
__device__ __forceinline__ int code_parts(int M) {
    return code_words(MW) == 0 ? M : (MW > 0 ? 4 : 2) * code_words(MW);
}
typedef float pair_ends __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const pair_ends lds_cends;
__device__ __forceinline__ float pair_lambda_term(int M, int stride, int m, uint32_t pair, uint32_t level) {
    const pair_ends e = *reinterpret_cast<lds_cends*>((uintptr_t)(pair * 8u + (uint32_t)(m * stride * 8)));     // (the table lies at address 0)
    const float c2 = *reinterpret_cast<lds_cfloat*>((uintptr_t)(pair * 4u + (uint32_t)(M * stride * 8 + m * stride * 4)));
    const float lam = fmaf((float)level, 0.0625f, -6.0f);
    return fmaf(fmaf(lam, lam, -lam), c2, fmaf(lam, e.y, e.x));
}
typedef uint32_t code_piece __attribute__((ext_vector_type(4), aligned(2)));      // eight sub-parts of a code
__device__ __forceinline__ void put_pair(float* lut, int M, int stride, int m, int pair, float b2, float d2, float c2) {
    reinterpret_cast<float2*>(lut)[m * stride + pair] = make_float2(b2, d2);
    lut[(2 * M + m) * stride + pair] = c2;
}

// Scores U candidate positions per thread (wb + u * 64 + lane: a wavefront walks its own contiguous
// piece of the candidate list, U windows of 64 positions at a time) and leaves their keys (ordered
// score bits) in key[0..U).  CHECK: positions may reach pend (their keys are left alone).
// RUNS: every thread searches the run list (short runs), the wavefront walks it (long ones) or marks it (between).
template <int MW, int U, bool CHECK, bool TAPS, int RUNS>
__device__ __forceinline__ void score_batch(const RerankArgs& g, int64_t q, int wb, int lane, int pend,
                                            const float* lut, uint32_t* key, const RunList& R, WaveRuns& wr, MarkedRuns& mr,
                                            uint32_t marks, RunCursor& cur, uint32_t& kmin, uint32_t& kmax) {
    const int p0 = wb + lane;
    constexpr int NW = code_words(MW);                         // code words fetched up front
    const int M = code_parts<MW>(g.M);
    uint32_t src[U];
    uint32_t cw[U][NW > 0 ? NW : 1];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t p = (uint32_t)(p0 + u * kWave);
        if (RUNS == kMarkRuns) {
            constexpr int G = U < 4 ? U : 4;                   // windows marked together
            if (u % G == 0) mr.group(R, (uint32_t)(wb + u * kWave), G * kWave, lane, marks);
            const bool wanted = !CHECK || p < (uint32_t)pend;
            const uint32_t delta = mr.window(R, p, wanted, u % G, lane, marks);
            src[u] = wanted ? p + delta
                            : (uint32_t)__builtin_amdgcn_readlane((int)(mr.v_start + mr.v_delta), 0);   // as below
        } else if (RUNS == kWalkRuns) {
            const uint32_t delta = wr.window(R, (uint32_t)(wb + u * kWave), lane);
            // a position past the end reads the first candidate of a run the wavefront holds
            src[u] = (!CHECK || p < (uint32_t)pend) ? p + delta : (uint32_t)__builtin_amdgcn_readlane((int)wr.v_src, 0);
        } else if (!CHECK || p < (uint32_t)pend) {
            if (p >= cur.next_start) {
                // usually the next run; otherwise the run is found by halving what is left of the list
                // (a thread's first position, or short runs: a step of 64 positions passes several)
                int lo = cur.run + 1;
                uint32_t next = R.start_at(lo + 1);
                if (p >= next) {
                    int hi = R.nr;                                  // start_at(lo) <= p < start_at(hi) = nc
                    ++lo;
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        const bool ge = R.start_at(mid) <= p;
                        lo = ge ? mid : lo;
                        hi = ge ? hi : mid;
                    }
                    next = R.start_at(lo + 1);
                }
                cur.run = lo;
                cur.next_start = next;
                cur.delta = R.src_at(lo) - R.start_at(lo);
            }
            src[u] = p + cur.delta;
        } else {
            src[u] = R.src_at(0);
        }
    }
    if (NW > 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t* c = reinterpret_cast<const uint32_t*>(g.codes + (size_t)src[u] * (4 * NW));
            if (NW == 2) {
                const uint2 v = *reinterpret_cast<const uint2*>(c);
                cw[u][0] = v.x;
                cw[u][NW > 1 ? 1 : 0] = v.y;
            } else if (NW == 4) {
                const uint4 v = *reinterpret_cast<const uint4*>(c);
                cw[u][0] = v.x;
                cw[u][NW > 1 ? 1 : 0] = v.y;
                cw[u][NW > 2 ? 2 : 0] = v.z;
                cw[u][NW > 3 ? 3 : 0] = v.w;
            } else {
#pragma unroll
                for (int j = 0; j < NW; ++j) cw[u][j] = c[j];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int p = p0 + u * kWave;
        if (CHECK && p >= pend) continue;
        float s;
        if (MW > 0) {
            s = lut_at_byte<0>(0, cw[u][0]);               // sum in ascending m
            s += lut_at_byte<1>(1, cw[u][0]);
            s += lut_at_byte<2>(2, cw[u][0]);
            s += lut_at_byte<3>(3, cw[u][0]);
#pragma unroll
            for (int j = 1; j < MW; ++j) {
                const uint32_t wv = cw[u][j];
                s += lut_at_byte<0>(j * 4 + 0, wv);
                s += lut_at_byte<1>(j * 4 + 1, wv);
                s += lut_at_byte<2>(j * 4 + 2, wv);
                s += lut_at_byte<3>(j * 4 + 3, wv);
            }
        } else if (MW < 0 && NW > 0) {
            // two bytes per sub-part, two sub-parts per word
            s = 0.0f;
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                const uint32_t wv = cw[u][j];
                s += pair_lambda_term(M, g.pair_stride, 2 * j, wv & 0xffu, (wv >> 8) & 0xffu);
                s += pair_lambda_term(M, g.pair_stride, 2 * j + 1, (wv >> 16) & 0xffu, wv >> 24);
            }
        } else if (MW < 0) {
            const uint16_t* code = reinterpret_cast<const uint16_t*>(g.codes) + (size_t)src[u] * M;
            s = 0.0f;
            int m = 0;
            auto pieces = [&](auto count) {                    // asked for together
                constexpr int n = decltype(count)::value;
                code_piece v[n];
#pragma unroll
                for (int i = 0; i < n; ++i) v[i] = *reinterpret_cast<const code_piece*>(code + m + 8 * i);
#pragma unroll
                for (int i = 0; i < 4 * n; ++i) {
                    const uint32_t wv = v[i / 4][i % 4];
                    s += pair_lambda_term(M, g.pair_stride, m + 2 * i, wv & 0xffu, (wv >> 8) & 0xffu);
                    s += pair_lambda_term(M, g.pair_stride, m + 2 * i + 1, (wv >> 16) & 0xffu, wv >> 24);
                }
                m += 8 * n;
            };
            if constexpr (MW == kPairLong) {
                while (m + 32 <= M) pieces(std::integral_constant<int, 4>{});
                if (m + 16 <= M) pieces(std::integral_constant<int, 2>{});
            }
            while (m + 8 <= M) pieces(std::integral_constant<int, 1>{});
#pragma unroll 2
            for (; m < M; ++m) s += pair_lambda_term(M, g.pair_stride, m, code[m] & 0xffu, code[m] >> 8);
        } else {
            const uint8_t* code = g.codes + (size_t)src[u] * M;
            s = 0.0f;
            for (int m = 0; m < M; ++m) s += lut[m * 256 + code[m]];
        }
        const uint32_t ky = mono_key(s);
        key[u] = ky;
        kmin = min(kmin, ky);
        kmax = max(kmax, ky);
        if (TAPS) {
            if (g.scores) g.scores[(size_t)q * g.C + p] = s;
            if (g.cand_ids) g.cand_ids[(size_t)q * g.C + p] = (int64_t)g.ids[src[u]];
        }
    }
}

// MW = 32-bit words per code (M/4) for M in {4, 8, 12, 16, 32}; 0 = any other M (byte loads);
// MW < 0 = codes hold (centroid pair, lambda level) per sub-part, scored by Eq. 9 directly.
// LONG: results may outnumber the workgroup's threads (apart, because that end costs the usual lists 1 % in the kernel that
// ranks as well).
// Query q, whose run list of meta.x runs and meta.y candidates is in g.runs.  MARKS: runs of medium length are marked (the kernel
// that ranks the head pass's left-over queries has no registers to spare for that).  READY: the level-1 distances, the table of Eq. 9
// and the first runs are in LDS, the histogram is zero.  (Arguments by value: by reference the kernels for pair codes of two and four
// words spilled, 5 to 8 % slower.)
template <int MW, bool TAPS, bool MARKS, bool LONG, bool READY>
__device__ __forceinline__ void rerank_query(const RerankArgs g, const RerankLds L, int64_t q, uint2 meta, unsigned char* smem) {
    unsigned long long* surv = reinterpret_cast<unsigned long long*>(smem + L.surv);
    float* lut = reinterpret_cast<float*>(smem);                 // L.lut == 0
    float* sa = reinterpret_cast<float*>(smem + L.a);
    uint32_t* run_src = reinterpret_cast<uint32_t*>(smem + L.run_src);
    uint32_t* run_start = reinterpret_cast<uint32_t*>(smem + L.run_start);
    uint32_t* hist = reinterpret_cast<uint32_t*>(smem + L.hist);
    uint32_t* part = reinterpret_cast<uint32_t*>(smem + L.part);
    uint32_t* misc = reinterpret_cast<uint32_t*>(smem + L.misc);

    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & (kWave - 1);
    const int M = g.M, k1 = g.k1, T = g.T, k = g.k;
    const int nlut = M * 256;
    const uint2* qruns = g.runs + (size_t)q * T;

    // ---- issue every load that needs no other result first ------------------------------------------
    uint2 run0 = make_uint2(0u, 0u);
    if (!READY && tid < kRunPrefetch && tid < L.rcap) run0 = qruns[tid];
    // table entries: a thread takes code value c = tid mod 256 of the sub-parts m0, m0 + ms, ... (m0 and ms
    // are the same for a wavefront, so which sub-parts exist is decided by scalar code)
    const int lut_c = tid & 255;
    const int lut_m0 = __builtin_amdgcn_readfirstlane(tid >> 8), lut_ms = nt >> 8;
    const int Mlut = code_parts<MW>(M);
    // entries a thread fetches per round: with codes of up to eight bytes all of a thread's entries at once, so
    // that no load is waited for inside the table phase (256 threads had two rounds of four)
    constexpr int kEnt = (MW > 0 && MW <= 2) ? 8 : 4;
    constexpr bool kOneRound = MW > 0 && 4 * MW <= kEnt;
    CodeEntry ent[kEnt];
    if (!READY) {
#pragma unroll
        for (int u = 0; u < kEnt; ++u) {
            const int m = lut_m0 + u * lut_ms;
            ent[u] = g.table[(m < Mlut ? m : 0) * 256 + lut_c];
        }
        for (int e = tid; e < M * k1; e += nt) sa[e] = g.a[(size_t)q * M * k1 + e];
        for (int e = tid; e < kHistSize; e += nt) hist[e] = 0;
    }
    const int nr = __builtin_amdgcn_readfirstlane((int)meta.x);     // the same in every thread
    const int nc = __builtin_amdgcn_readfirstlane((int)meta.y);
    int steps = 0;
    while ((1 << steps) < nr) ++steps;
    const int nr_lds = nr < L.rcap ? nr : L.rcap;
    if (!READY && tid < kRunPrefetch && tid < nr_lds) {
        run_src[tid] = run0.x;
        run_start[tid] = run0.y;
    }
    for (int r = kRunPrefetch + tid; !READY && r < nr_lds; r += nt) {
        const uint2 run = qruns[r];
        run_src[r] = run.x;
        run_start[r] = run.y;
    }
    if (tid == 0) {
        if (nr <= L.rcap) run_start[nr] = (uint32_t)nc;
        misc[kMin] = 0xffffffffu;
        misc[kMax] = 0u;
        misc[kNumSurv] = 0u;
        if (LONG) misc[kFullBin] = 0u;
    }
    RunList R;
    R.src = L.run_src; R.start = L.run_start; R.mem = qruns; R.rcap = L.rcap; R.nr = nr; R.nc = (uint32_t)nc;
    __syncthreads();

    // ---- LUT of Eq. 9 summands ------------------------------------------------------------------------
    auto table_entry = [&](int m, const CodeEntry& ce) {
        const int e = m * 256 + lut_c;
        const float* sam = sa + m * k1;
        const float b2 = sam[ce.ij & 0xffu];
        const float a2 = sam[(ce.ij >> 8) & 0xffu];
        if (MW < 0) {
            // entry = centroid pair number; its kc field holds c^2
            if (lut_c < g.pair_stride) put_pair(lut, Mlut, g.pair_stride, m, lut_c, b2, a2 - b2, ce.kc);
            return;
        }
        // Eq. 9 rearranged: b^2 + lam (a^2 - b^2) + (lam^2 - lam) c^2, the last term folded per code value
        const float v = fmaf(ce.lam, a2 - b2, b2) + ce.kc;
        lut[e] = v;
        if (TAPS && g.lut) g.lut[(size_t)q * nlut + e] = v;
    };
    if constexpr (READY) {
    } else if constexpr (kOneRound) {
#pragma unroll
        for (int u = 0; u < kEnt; ++u) {
            const int m = lut_m0 + u * lut_ms;
            if (m < Mlut) table_entry(m, ent[u]);
        }
    } else {
        for (int mb = lut_m0; mb < Mlut; mb += 4 * lut_ms) {
            CodeEntry cur_ent[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) cur_ent[u] = ent[u];
            if (mb + 4 * lut_ms < Mlut) {          // the next round's entries are fetched while this one is worked on
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int m = mb + (4 + u) * lut_ms;
                    ent[u] = g.table[(m < Mlut ? m : 0) * 256 + lut_c];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int m = mb + u * lut_ms;
                if (m < Mlut) table_entry(m, cur_ent[u]);      // (no early exit: the loop must unroll in full)
            }
        }
    }
    if (!READY) __syncthreads();

    // ---- scores: wavefront v owns positions [v * chunk, (v + 1) * chunk); position pos0 + u * 64 -> key[u] -----
    const int chunk = ((nc + (nt >> 6) - 1) / (nt >> 6) + kWave - 1) & ~(kWave - 1);     // <= 64 * kKeysPerThread
    const int pos0 = (tid >> 6) * chunk + lane;
    const int pend = min(nc, ((tid >> 6) + 1) * chunk);      // this wavefront's positions end here
    uint32_t key[kKeysPerThread];
#pragma unroll
    for (int u = 0; u < kKeysPerThread; ++u) key[u] = 0xffffffffu;
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    if (nc > 0) {
        const int wbase = __builtin_amdgcn_readfirstlane(pos0 - lane);    // the same for a wavefront
        // eight positions in flight per thread; four when a code has four or more words or holds (pair, lambda)
        // tuples, whose scoring needs the registers, two of sixteen words
        constexpr int UB = MW == -16 ? 2 : ((MW >= 4 || MW <= -2) ? 4 : 8);
        static_assert(kKeysPerThread % 4 == 0, "batches of two, four or eight");
        WaveRuns wr;
        MarkedRuns mr;                         // (not in the kernel that ranks as well)
        const uint32_t marks = L.part + (uint32_t)(tid & ~(kWave - 1)) * 4u;      // 256 bytes a wavefront: its words of part[]
        RunCursor cur;                         // positions of a thread only grow
        auto score_all = [&](auto how) {
            constexpr int RUNS = decltype(how)::value;
#pragma unroll
            for (int b = 0; b * UB + UB <= kKeysPerThread; ++b) {
                const int base = wbase + b * UB * kWave;
                if (base + UB * kWave <= pend)
                    score_batch<MW, UB, false, TAPS, RUNS>(g, q, base, lane, pend, lut, key + b * UB, R, wr, mr, marks, cur, kmin, kmax);
                else if (base < pend)
                    score_batch<MW, UB, true, TAPS, RUNS>(g, q, base, lane, pend, lut, key + b * UB, R, wr, mr, marks, cur, kmin, kmax);
            }
            if (kKeysPerThread % UB) {         // a last batch of four
                constexpr int done = kKeysPerThread / UB * UB;
                const int base = wbase + done * kWave;
                if (base + 4 * kWave <= pend)
                    score_batch<MW, 4, false, TAPS, RUNS>(g, q, base, lane, pend, lut, key + done, R, wr, mr, marks, cur, kmin, kmax);
                else if (base < pend)
                    score_batch<MW, 4, true, TAPS, RUNS>(g, q, base, lane, pend, lut, key + done, R, wr, mr, marks, cur, kmin, kmax);
            }
        };
        if (MARKS && nr * kMarkMinRun <= nc && nr * kMarkMaxRun > nc) {
            mr.load(R, 0, lane);
            score_all(std::integral_constant<int, kMarkRuns>{});
        } else if (nr * kWalkMinRun <= nc) {   // runs long enough that a window of 64 positions meets few of them
            wr.seek(R, (uint32_t)wbase, lane);
            score_all(std::integral_constant<int, kWalkRuns>{});
        } else {
            cur.run = 0;
            cur.next_start = R.start_at(1);
            cur.delta = R.src_at(0) - R.start_at(0);
            score_all(std::integral_constant<int, kSearchRuns>{});
        }
    }
    if (TAPS && g.n_cand && tid == 0) g.n_cand[q] = (uint32_t)nc;
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if (lane == 0) {
        atomicMin(&misc[kMin], kmin);
        atomicMax(&misc[kMax], kmax);
    }
    __syncthreads();

    // ---- the k smallest (score, id): (key, position) of a superset of the answer -> surv ---------------
    const int kk = k < nc ? k : nc;           // results that exist
    int nsurv;
    bool by_bin = false;                       // the survivors can be placed by their histogram bin (see below)
    uint32_t lo_key = 0;
    int shift = 0;
    if (nc <= L.scap) {                        // few candidates: order all of them
#pragma unroll
        for (int u = 0; u < kKeysPerThread; ++u) {
            const int p = pos0 + u * kWave;
            if (p < pend) surv[p] = ((unsigned long long)key[u] << 32) | (uint32_t)p;
        }
        nsurv = nc;
    } else {
        lo_key = misc[kMin];
        const uint32_t range = misc[kMax] - lo_key;
        const int width = 32 - __clz((int)(range | 1u));           // bits needed for range
        shift = width > kHistBits ? width - kHistBits : 0;          // (key - lo_key) >> shift < 1024
#pragma unroll
        for (int u = 0; u < kKeysPerThread; ++u) {
            if (u * kWave >= chunk) break;                             // same for the whole workgroup
            if (pos0 + u * kWave < pend) atomicAdd(&hist[(key[u] - lo_key) >> shift], 1u);
        }
        __syncthreads();
        // counts -> first positions, in place (a prefix sum by the whole workgroup); the thread that owns the
        // bin bsel with count(< bsel) < kk <= count(<= bsel) notes it
        {
            const int bpt = kHistSize / nt;                        // 4, 2 or 1 bins per thread
            uint32_t sum = 0;
            for (int j = 0; j < bpt; ++j) sum += hist[tid * bpt + j];
            uint32_t total;
            uint32_t c = block_exclusive_sum(sum, part, total);
            for (int j = 0; j < bpt; ++j) {
                const uint32_t cnt = hist[tid * bpt + j];
                hist[tid * bpt + j] = c;
                if (LONG && k > nt && c < (uint32_t)kk && cnt > (uint32_t)kBinRankMax) misc[kFullBin] = 1u;
                if (c < (uint32_t)kk && (uint32_t)kk <= c + cnt) {
                    misc[kSel] = (uint32_t)(tid * bpt + j);
                    misc[kSelCount] = c + cnt;
                }
                c += cnt;
            }
        }
        __syncthreads();
        const uint32_t bsel = misc[kSel];
        const uint32_t count_le = misc[kSelCount];
        if (count_le <= (uint32_t)L.scap) {
            // keys of the bins <= bsel are the keys <= thr
            const unsigned long long thr64 = (unsigned long long)lo_key + (((unsigned long long)bsel + 1ull) << shift) - 1ull;
            const uint32_t thr = thr64 > 0xffffffffull ? 0xffffffffu : (uint32_t)thr64;
            // (long lists: a bin of many, ties, would keep its threads long; those are sorted)
            by_bin = thr != 0xffffffffu && (count_le <= (uint32_t)nt || (LONG && k > nt && count_le <= (uint32_t)(kSurvPer * nt) && misc[kFullBin] == 0u));
            if (thr != 0xffffffffu) {
                // key slots without a candidate hold 0xffffffff > thr.  A wavefront counts its keys <= thr,
                // reserves room for them with one atomic, then writes them: no wait for LDS per window
                uint32_t mine = 0;
#pragma unroll
                for (int u = 0; u < kKeysPerThread; ++u) mine += (uint32_t)__popcll(__ballot(key[u] <= thr));
                uint32_t at = 0;
                if (lane == 0 && mine) at = atomicAdd(&misc[kNumSurv], mine);
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
                for (int u = 0; u < kKeysPerThread; ++u) {
                    const unsigned long long hm = __ballot(key[u] <= thr);
                    if (hm == 0ull) continue;                          // the same for the wavefront
                    if (key[u] <= thr) {
                        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(hm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hm, 0u));
                        surv[at + below] = ((unsigned long long)key[u] << 32) | (uint32_t)(pos0 + u * kWave);
                    }
                    at += (uint32_t)__popcll(hm);
                }
            } else {
#pragma unroll
                for (int u = 0; u < kKeysPerThread; ++u) {
                    const int p = pos0 + u * kWave;
                    if (u * kWave >= chunk) break;
                    if (p < pend && key[u] <= thr)
                        surv[atomicAdd(&misc[kNumSurv], 1u)] = ((unsigned long long)key[u] << 32) | (uint32_t)p;
                }
            }
            nsurv = (int)count_le;
        } else {
            // exact selection: k-th smallest score key, then (only if that score is tied) the ids
            uint32_t* rout = misc + kRadix;
            uint32_t prefix = 0, mask = 0, need = (uint32_t)kk, bucket = 0;
            const int shifts[4] = {22, 12, 2, 0};
            const int nbits[4] = {10, 10, 10, 2};
            __syncthreads();
            for (int pass = 0; pass < 4; ++pass) {
                radix_select_pass(prefix, mask, shifts[pass], nbits[pass], need, hist, part, rout, [&](auto f) {
#pragma unroll
                    for (int u = 0; u < kKeysPerThread; ++u)
                        if (pos0 + u * kWave < pend) f(key[u]);
                });
                prefix |= rout[0] << shifts[pass];
                mask |= ((1u << nbits[pass]) - 1u) << shifts[pass];
                need = rout[1];
                bucket = rout[2];
                __syncthreads();
            }
            const uint32_t tau = prefix;
            uint32_t id_cut = 0xffffffffu;     // among candidates with key == tau keep ids <= id_cut
            if (need < bucket) {
                uint32_t iprefix = 0, imask = 0;
                for (int pass = 0; pass < 4; ++pass) {
                    radix_select_pass(iprefix, imask, shifts[pass], nbits[pass], need, hist, part, rout, [&](auto f) {
#pragma unroll
                        for (int u = 0; u < kKeysPerThread; ++u) {
                            const int p = pos0 + u * kWave;
                            if (p < pend && key[u] == tau) f(g.ids[source_of((uint32_t)p, steps, R)]);
                        }
                    });
                    iprefix |= rout[0] << shifts[pass];
                    imask |= ((1u << nbits[pass]) - 1u) << shifts[pass];
                    need = rout[1];
                    __syncthreads();
                }
                id_cut = iprefix;
            }
#pragma unroll
            for (int u = 0; u < kKeysPerThread; ++u) {
                const int p = pos0 + u * kWave;
                if (p >= pend || key[u] > tau) continue;
                if (key[u] == tau && id_cut != 0xffffffffu && g.ids[source_of((uint32_t)p, steps, R)] > id_cut) continue;
                surv[atomicAdd(&misc[kNumSurv], 1u)] = ((unsigned long long)key[u] << 32) | (uint32_t)p;
            }
            nsurv = kk;
        }
    }
    __syncthreads();

    // ---- usual case: the survivors are placed by their histogram bin, no sort -----------------------------
    // hist[] holds the first position of every bin among the sorted keys.  A thread takes one survivor,
    // fetches its id, and drops the (score bits, id) key into its bin's range with one LDS atomic; then every
    // key counts the smaller keys of its own bin (one to four entries) and that is its place in the output.
    if (by_bin && nsurv <= nt) {
        const bool have = tid < nsurv;
        unsigned long long mine = ~0ull;
        uint32_t bin = 0;
        if (have) {
            const unsigned long long kp = surv[tid];
            mine = (kp & 0xffffffff00000000ull) | g.ids[source_of((uint32_t)kp, steps, R)];
            bin = ((uint32_t)(kp >> 32) - lo_key) >> shift;
        }
        __syncthreads();                       // every surv[] entry has been read
        if (have) surv[atomicAdd(&hist[bin], 1u)] = mine;
        __syncthreads();                       // hist[b] is now the end of bin b, the start of bin b + 1
        if (have) {
            const uint32_t first = bin ? hist[bin - 1] : 0u, end = hist[bin];
            uint32_t r = first;
            for (uint32_t x = first; x < end; ++x) r += surv[x] < mine ? 1u : 0u;
            if (r < (uint32_t)kk) {
                g.out_ids[(size_t)q * k + r] = (int64_t)(uint32_t)mine;
                g.out_dists[(size_t)q * k + r] = mono_inv((uint32_t)(mine >> 32));
            }
        }
        for (int e = kk + tid; e < k; e += nt) {
            g.out_ids[(size_t)q * k + e] = (int64_t)-1;
            g.out_dists[(size_t)q * k + e] = __builtin_inff();
        }
        return;
    }

    // ---- long result lists: the same with up to eight survivors a thread, and the output written in order -------------
    // (1,000 results of 4,096 candidates, 10,000 queries: 243 us; sorting 2,048 keys with 256 threads 309)
    if (LONG && by_bin && g.set_only) {
        // Their order is of no use to the caller, nor are their distances: what lies below the k-th's bin goes out as it comes, a
        // wavefront's results side by side, and of that bin those are counted out that still belong
        // (1,000 of 4,096, 10,000 queries: 165 us instead of 200).
        static_assert(2 * kBinRankMax <= 256, "the bin's keys take the place of part[]");
        unsigned long long* edge = reinterpret_cast<unsigned long long*>(part);
        const uint32_t bsel = misc[kSel], lower = hist[bsel];  // (first positions)
        if (tid == 0) misc[kRadix] = misc[kRadix + 1] = 0u;
        __syncthreads();
        uint32_t id[kSurvPer], bits[kSurvPer];
#pragma unroll
        for (int s = 0; s < kSurvPer; ++s) {
            if (s * nt >= nsurv) break;                // the same for the whole workgroup
            const int e = tid + s * nt;
            const unsigned long long kp = surv[e < nsurv ? e : 0];
            bits[s] = (uint32_t)(kp >> 32);
            id[s] = g.ids[source_of((uint32_t)kp, steps, R)];
        }
#pragma unroll
        for (int s = 0; s < kSurvPer; ++s) {
            if (s * nt >= nsurv) break;
            const bool have = tid + s * nt < nsurv;
            const uint32_t bin = (bits[s] - lo_key) >> shift;
            const unsigned long long low = __ballot(have && bin < bsel);
            uint32_t at = 0;
            if (lane == 0 && low) at = atomicAdd(&misc[kRadix], (uint32_t)__popcll(low));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(low & ((1ull << lane) - 1ull));
            if (have && bin < bsel) g.out_ids[(size_t)q * k + at] = (int64_t)id[s];
            if (have && bin == bsel) edge[atomicAdd(&misc[kRadix + 1], 1u)] = ((unsigned long long)bits[s] << 32) | id[s];
        }
        __syncthreads();
        const uint32_t nedge = misc[kRadix + 1];
        if (tid < (int)nedge) {
            const unsigned long long mine = edge[tid];
            uint32_t r = lower;
            for (uint32_t x = 0; x < nedge; ++x) r += edge[x] < mine ? 1u : 0u;
            if (r < (uint32_t)kk) g.out_ids[(size_t)q * k + r] = (int64_t)(uint32_t)mine;
        }
        for (int e = kk + tid; e < k; e += nt) g.out_ids[(size_t)q * k + e] = (int64_t)-1;
        return;
    }
    if (LONG && by_bin) {
        unsigned long long mine[kSurvPer];
        uint32_t at[kSurvPer];
#pragma unroll
        for (int s = 0; s < kSurvPer; ++s) {
            if (s * nt >= nsurv) break;                // the same for the whole workgroup
            const int e = tid + s * nt;
            mine[s] = ~0ull;
            if (e < nsurv) {
                const unsigned long long kp = surv[e];
                mine[s] = (kp & 0xffffffff00000000ull) | g.ids[source_of((uint32_t)kp, steps, R)];
            }
        }
        auto bin_of = [&](unsigned long long key) { return ((uint32_t)(key >> 32) - lo_key) >> shift; };
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kSurvPer; ++s) {
            if (s * nt >= nsurv) break;
            if (tid + s * nt < nsurv) surv[atomicAdd(&hist[bin_of(mine[s])], 1u)] = mine[s];
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kSurvPer; ++s) {
            if (s * nt >= nsurv) break;
            if (tid + s * nt >= nsurv) continue;
            const uint32_t bin = bin_of(mine[s]);
            const uint32_t first = bin ? hist[bin - 1] : 0u, end = hist[bin];
            at[s] = first;
            for (uint32_t x = first; x < end; ++x) at[s] += surv[x] < mine[s] ? 1u : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kSurvPer; ++s) {
            if (s * nt >= nsurv) break;
            if (tid + s * nt < nsurv) surv[at[s]] = mine[s];
        }
        __syncthreads();
        for (int e = tid; e < k; e += nt) {
            const unsigned long long skey = surv[e < kk ? e : 0];
            g.out_ids[(size_t)q * k + e] = e < kk ? (int64_t)(uint32_t)skey : (int64_t)-1;
            g.out_dists[(size_t)q * k + e] = e < kk ? mono_inv((uint32_t)(skey >> 32)) : __builtin_inff();
        }
        return;
    }

    // ---- otherwise: fetch the survivors' ids: 64-bit keys (score bits, id) ------------------------------
    // (one round of loads for the whole list: the thread that holds a surviving key does not fetch the id
    // itself, or a wavefront would wait for memory once per key slot)
    for (int e = tid; e < nsurv; e += nt) {
        const unsigned long long kp = surv[e];
        const uint32_t id = g.ids[source_of((uint32_t)kp, steps, R)];
        surv[e] = (kp & 0xffffffff00000000ull) | id;
    }
    __syncthreads();

    // ---- order the survivors, write the first k ---------------------------------------------------------
    if (nsurv <= kCountRankMax) {
        // a handful: rank = number of smaller keys (keys are unique); four adjacent lanes share one survivor
        const int sub = tid & 3;
        for (int e0 = 0; e0 < nsurv; e0 += nt / 4) {
            const int e = e0 + (tid >> 2);
            const bool valid = e < nsurv;
            const unsigned long long skey = valid ? surv[e] : 0ull;
            uint32_t rank = 0;
            for (int j = sub; j < nsurv; j += 4) rank += (surv[j] < skey) ? 1u : 0u;
            rank += quad_swap1(rank);
            rank += quad_swap2(rank);
            if (valid && sub == 0 && rank < (uint32_t)k) {
                g.out_ids[(size_t)q * k + rank] = (int64_t)(uint32_t)skey;
                g.out_dists[(size_t)q * k + rank] = mono_inv((uint32_t)(skey >> 32));
            }
        }
    } else {
        // sorted in registers, 64 keys per wavefront (comparisons grow as n log^2 n, not n^2)
        const int npad = next_pow2(nsurv) < kWave ? kWave : next_pow2(nsurv);
        for (int e = nsurv + tid; e < npad; e += nt) surv[e] = ~0ull;
        if (npad <= 4 * nt) block_sort_lds<4>(surv, npad, tid, nt);
        else bitonic_sort_lds(surv, npad, tid, nt);            // more than four keys per thread: all in LDS
        for (int e = tid; e < kk; e += nt) {
            const unsigned long long skey = surv[e];
            g.out_ids[(size_t)q * k + e] = (int64_t)(uint32_t)skey;
            g.out_dists[(size_t)q * k + e] = mono_inv((uint32_t)(skey >> 32));
        }
    }
    for (int e = kk + tid; e < k; e += nt) {
        g.out_ids[(size_t)q * k + e] = (int64_t)-1;
        g.out_dists[(size_t)q * k + e] = __builtin_inff();
    }
}

// FUSED: a query whose meta.x is kMetaTodo (the ranking head pass could not finish it) is first
// ranked in full by this workgroup.
template <int MW, bool TAPS, bool FUSED, bool LONG>
__global__ __launch_bounds__(1024, TAPS ? 1 : ((MW >= 8 || MW <= -6) ? 4 : 8)) void rerank_kernel(RerankArgs g, RerankLds L, RankArgs rk, RankOffsets RL) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t* misc = reinterpret_cast<uint32_t*>(smem + L.misc);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    int64_t q;
    uint2 meta;
    if ((int)blockIdx.x < g.early) {           // one of the queries the head pass left unfinished, if any
        if (blockIdx.x >= *g.todo_count) return;
        q = (int64_t)g.todo[blockIdx.x];
        meta = g.meta[q];
    } else {
        q = (int64_t)blockIdx.x - g.early;
        meta = g.meta[q];
        if (g.early > 0 && meta.x == kMetaTodo && meta.y < (uint32_t)g.early) return;   // an early workgroup has it
    }
    if (FUSED && meta.x == kMetaTodo) {        // same for the whole workgroup
        // the run list goes to memory (this query's own rows), the counts come back through LDS.
        // First the head pass's third level (128 tuples) by the first wavefront alone: few vector
        // instructions, and nearly every left-over query is finished by it; the full ranking by the
        // whole workgroup only if even those runs do not fill the candidate budget.
        bool ranked = false;
        if (g.mid_T1 > 0) {
            if (tid < kWave) {
                HeadLds& S = *reinterpret_cast<HeadLds*>(smem);
                const int R1 = rk.R < kHeadT ? rk.R : kHeadT;
                head_load_lists(rk, S, q, lane, R1);
                unsigned long long carry = ~0ull;
                const int r = head_level<2, true>(rk, S, q, lane, R1, g.mid_T1, 0, g.mid_npairs, RL.Tcap, true, carry, misc + kRanked);
                if (lane == 0) misc[kRanked + 2] = r == 1 ? 1u : 0u;
            }
            __syncthreads();
            ranked = misc[kRanked + 2] != 0u;
            __syncthreads();
        }
        if (!ranked) rank_query<2, true, kFusedPer, 0>(rk, RL, q, smem, misc + kRanked);
        meta = make_uint2(misc[kRanked], misc[kRanked + 1]);
    }
    rerank_query<MW, TAPS, !FUSED, LONG, false>(g, L, q, meta, smem);
}

// The table of Eq. 9 summands (see rerank_query) by the threads from `first` on, and the histogram cleared.
template <int MW>
__device__ __forceinline__ void prepare_table(const RerankArgs& g, const RerankLds& L, unsigned char* smem, int first) {
    float* lut = reinterpret_cast<float*>(smem);
    const float* sa = reinterpret_cast<const float*>(smem + L.a);
    uint32_t* hist = reinterpret_cast<uint32_t*>(smem + L.hist);
    const int who = (int)threadIdx.x - first, n = (int)blockDim.x - first;
    const int M = code_parts<MW>(g.M), per = MW < 0 ? g.pair_stride : 256, entries = M * per;
    constexpr int U = 4;                       // entries asked for together
    // the sub-part of an entry: half an entry from the next whole number, which is more than the product is off
    const float inv = 1.0f / (float)per;
    auto part_of = [&](int e) { return MW < 0 ? (int)(((float)e + 0.5f) * inv) : e / per; };
    for (int e0 = who; e0 < entries; e0 += U * n) {
        CodeEntry ent[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = min(e0 + u * n, entries - 1), m = part_of(e);
            ent[u] = g.table[m * 256 + (e - m * per)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * n;
            if (e >= entries) break;
            const int m = part_of(e);
            const float* sam = sa + m * g.k1;
            const float b2 = sam[ent[u].ij & 0xffu], a2 = sam[(ent[u].ij >> 8) & 0xffu];
            if (MW < 0) put_pair(lut, M, per, m, e - m * per, b2, a2 - b2, ent[u].kc);
            else lut[e] = fmaf(ent[u].lam, a2 - b2, b2) + ent[u].kc;
        }
    }
    for (int e = who; e < kHistSize; e += n) hist[e] = 0;
}

// The fixed bin order (rank_static_kernel has its definition) of a query whose lists are in LDS, by a workgroup: as many tuples at a
// time as it has threads.  part: two times 16 words for prefix sums.  Ends with a barrier.
__device__ __forceinline__ void rank_static_query(const RankArgs& g, const StaticOrder& so, int64_t q, const float* sLd, const uint32_t* sLid,
                                                  uint32_t* part, uint32_t* out_counts, const RunSink& sink) {
    const int tid = threadIdx.x, nt = blockDim.x, R = g.R;
    const uint32_t C = (uint32_t)g.C;
    const int r0 = R - 1 < kSlopeReferenceRank ? R - 1 : kSlopeReferenceRank;
    const float g1 = sLd[r0] - sLd[0], g2 = sLd[R + r0] - sLd[R];
    int slope = 0;
#pragma unroll
    for (int j = 0; j < kStaticSlopes - 1; ++j) slope += (g2 > so.thr[j] * g1) ? 1 : 0;
    const uint32_t* tab = so.table + (size_t)slope * so.Tn;
    uint32_t total = 0, nruns = 0;
    for (int base = 0; base < so.Tn && total < C; base += nt) {
        const int t = base + tid;
        uint32_t len = 0, o0 = 0;
        if (t < so.Tn) {
            const uint32_t ab = tab[t];
            const unsigned long long slot = (unsigned long long)sLid[ab >> 16] * g.k1k2 + sLid[R + (ab & 0xffffu)];
            o0 = g.offsets[slot];
            len = g.offsets[slot + 1] - o0;
        }
        uint32_t here, runs;
        const uint32_t start = total + block_exclusive_sum(len, part, here);
        const bool emit = len > 0 && start < C;
        const uint32_t at = nruns + block_exclusive_sum(emit ? 1u : 0u, part + 16, runs);
        if (emit && !sink.put(at, o0, start)) g.runs[(size_t)q * g.T + at] = make_uint2(o0, start);
        total += here;
        nruns += runs;
        __syncthreads();                       // (the prefix sums' memory)
    }
    if (tid == 0) {
        out_counts[0] = nruns;
        out_counts[1] = total < C ? total : C;
    }
    __syncthreads();
}

// A whole query of a small batch by one workgroup (1,024 threads, fewer where several share a compute unit), in one launch:
// traversal, ranking, re-ranking.  Every query has its compute unit, or a half or quarter of one, so what it costs is the chain of its
// steps, and of a launch that starts when the one before has drained (4 us each) there is one instead of three (one query
// 23.6 -> 20.6 us, 67 48.8 -> 37.3); lists, level-1 distances and runs stay in LDS, and the table of Eq. 9 is
// built while a wavefront per part sorts its list, if there is LDS for that and the ranking side by side.
template <int MW>
__global__ __launch_bounds__(1024, 4) void query_kernel(RerankArgs g, RerankLds L, RankArgs rk, RankOffsets RL, TraverseArgs tr, SmallQuery sm) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t* misc = reinterpret_cast<uint32_t*>(smem + L.misc);
    unsigned char* ranking = smem + sm.off_ranking;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int64_t q = blockIdx.x;
    float* sLd = reinterpret_cast<float*>(ranking + RL.Ld);
    uint32_t* sLid = reinterpret_cast<uint32_t*>(ranking + RL.Lid);
    uint8_t* tab = smem + sm.off_tables;
    if (sm.levels.T1[0] > 0)
        for (int e = tid; e < 2 * kHeadPairs / 4; e += (int)blockDim.x)
            reinterpret_cast<uint32_t*>(tab)[e] = e < kHeadPairs / 4 ? reinterpret_cast<const uint32_t*>(kHeadPairTable.a)[e]
                                                                     : reinterpret_cast<const uint32_t*>(kHeadPairTable.b)[e - kHeadPairs / 4];
    for (int e = tid; e < kPlaceBins; e += (int)blockDim.x) reinterpret_cast<uint32_t*>(ranking + RL.hist)[e] = 0u;
    traverse_one(tr, q, smem + sm.off_traverse, reinterpret_cast<float*>(smem + L.a), sLd, sLid,
                 [&](int first) {
                     if (!sm.late_table) prepare_table<MW>(g, L, smem, first);
                 });
    RunSink sink;
    sink.src = reinterpret_cast<uint32_t*>(smem + L.run_src);
    sink.start = reinterpret_cast<uint32_t*>(smem + L.run_start);
    sink.cap = (uint32_t)L.rcap;
    bool ranked = false;
    if (sm.fixed.table) {
        rank_static_query(rk, sm.fixed, q, sLd, sLid, reinterpret_cast<uint32_t*>(ranking + RL.part), misc + kRanked, sink);
        ranked = true;
    } else if (sm.levels.T1[0] > 0) {
        if (tid < kWave) {                     // the head pass's first two levels
            HeadLds& S = *reinterpret_cast<HeadLds*>(smem + sm.off_head);
            const int R1 = rk.R < kHeadT ? rk.R : kHeadT;
            for (int e = lane; e < R1; e += kWave) {
                S.A[e] = sLd[e];
                S.Aid[e] = sLid[e];
                S.B[e] = sLd[rk.R + e];
                S.Bid[e] = sLid[rk.R + e];
            }
            wave_lds_order();
            unsigned long long carry = ~0ull;
            int r = head_level<1, true>(rk, S, q, lane, R1, sm.levels.T1[0], 0, sm.levels.npairs[0], RL.Tcap, false, carry, misc + kRanked,
                                        tab, tab + kHeadPairs, sink);
            if (r == 0)
                r = head_level<1, true>(rk, S, q, lane, R1, sm.levels.T1[1], sm.levels.npairs[0], sm.levels.npairs[1], RL.Tcap, true, carry,
                                        misc + kRanked, tab, tab + kHeadPairs, sink);
            if (lane == 0) misc[kRanked + 2] = r == 1 ? 1u : 0u;
        }
        __syncthreads();
        ranked = misc[kRanked + 2] != 0u;
        __syncthreads();
    }
    if (!ranked) rank_query<0, true, 4, kRankPlace, true>(rk, RL, q, ranking, misc + kRanked, sink);
    if (sm.late_table) prepare_table<MW>(g, L, smem, 0);
    rerank_query<MW, false, true, true, true>(g, L, q, make_uint2(misc[kRanked], misc[kRanked + 1]), smem);
}


// ---- one translation unit per code width instantiates its kernels through these ------------------------------
// HAS_TAPS: a variant with the taps exists for this code width (the word-wise (pair, lambda) variants have none:
// the tapped call takes the byte-wise kernel).
template <int MW, bool HAS_TAPS>
inline hipError_t launch_rerank_variant(const RerankArgs& a, const RerankLds& L, const RankArgs& rk, const RankOffsets& RL,
                                        bool taps, bool fused, hipStream_t s) {
    const dim3 grid((unsigned)(a.nq + a.early)), block(a.threads);
    if (fused && a.k > a.threads) {
        hipLaunchKernelGGL((rerank_kernel<MW, false, true, true>), grid, block, L.total, s, a, L, rk, RL);
    } else if (fused) {
        hipLaunchKernelGGL((rerank_kernel<MW, false, true, false>), grid, block, L.total, s, a, L, rk, RL);
    } else if (taps) {
        if constexpr (HAS_TAPS) hipLaunchKernelGGL((rerank_kernel<MW, true, false, true>), grid, block, L.total, s, a, L, rk, RL);
        else return hipErrorInvalidValue;
    } else {
        hipLaunchKernelGGL((rerank_kernel<MW, false, false, true>), grid, block, L.total, s, a, L, rk, RL);
    }
    return hipGetLastError();
}

template <int MW>
inline hipError_t launch_query_variant(const RerankArgs& a, const RerankLds& L, const RankArgs& rk, const RankOffsets& RL, const TraverseArgs& tr,
                                       const SmallQuery& sm, hipStream_t s) {
    hipLaunchKernelGGL((query_kernel<MW>), dim3((unsigned)a.nq), dim3(a.threads), sm.lds, s, a, L, rk, RL, tr, sm);
    return hipGetLastError();
}

template <int MW, bool HAS_TAPS>
inline hipError_t configure_rerank_variant(size_t max_dynamic_lds) {
    const void* kernels[5] = {reinterpret_cast<const void*>(rerank_kernel<MW, false, false, true>),
                              reinterpret_cast<const void*>(rerank_kernel<MW, false, true, false>),
                              reinterpret_cast<const void*>(rerank_kernel<MW, false, true, true>),
                              reinterpret_cast<const void*>(query_kernel<MW>), nullptr};
    if constexpr (HAS_TAPS) kernels[4] = reinterpret_cast<const void*>(rerank_kernel<MW, true, false, true>);
    for (const void* kfn : kernels) {
        if (!kfn) continue;
        hipFuncAttributes attr;
        hipError_t e = hipFuncGetAttributes(&attr, kfn);
        if (e != hipSuccess) return e;
        if (attr.sharedSizeBytes != 0) return hipErrorInvalidValue;   // the LUT must start at LDS address 0
        e = hipFuncSetAttribute(kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_dynamic_lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

#define PQT_RERANK_VARIANT_DEFINE(NAME, MW, HAS_TAPS)                                                                       \
    hipError_t launch_rerank_##NAME(const RerankArgs& a, const RerankLds& L, const RankArgs& rk, const RankOffsets& RL,      \
                                    bool taps, bool fused, hipStream_t s) {                                                 \
        return launch_rerank_variant<MW, HAS_TAPS>(a, L, rk, RL, taps, fused, s);                                           \
    }                                                                                                                       \
    hipError_t launch_query_##NAME(const RerankArgs& a, const RerankLds& L, const RankArgs& rk, const RankOffsets& RL,       \
                                   const TraverseArgs& tr, const SmallQuery& sm, hipStream_t s) {                           \
        return launch_query_variant<MW>(a, L, rk, RL, tr, sm, s);                                                           \
    }                                                                                                                       \
    hipError_t configure_rerank_##NAME(size_t max_dynamic_lds) { return configure_rerank_variant<MW, HAS_TAPS>(max_dynamic_lds); }

}  // namespace pqt
