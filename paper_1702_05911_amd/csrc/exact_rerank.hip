// Exact re-ranking of a short list (step (3) of the pipelines in Sec. 1; the paper's PQT_2 of
// Table 1): the first k_short results of the line-quantisation re-ranking are scored again by their
// exact squared distance ||y - x||^2 to the raw database vectors, and the k best by (distance, id)
// are returned.
//
// One workgroup of 256 threads per query.  The query sits in LDS; a group of lanes (64, or fewer when
// the vector is short) reads one database row with consecutive 16-byte pieces per lane, so a row is a
// few fully used cache lines; four rows are on their way per group.  Bound by the memory system: k_short
// random rows of D elements per query.
// Squared differences are summed per lane in ascending dimension, then across the group by a fixed
// xor tree, so the result does not depend on scheduling.  The (ordered distance bits, id) keys stay in LDS; the k
// smallest are found by a 1024-bin histogram and placed by their bin (every key counts the smaller ones of its
// own bin), as in the re-ranking; where ties crowd a bin all are sorted.
// 10,000 queries, 1,000 rows of 128 bytes, k = 100: 199 us (6.4 TB/s of rows); with two rows on their way behind a load of their ids, and
// a sort of all 1,024 keys, 281.
#include "../../include/pqt.h"
#include "pqt_device.hpp"
#include "pqt_kernels.hpp"
#include "row_distance.hpp"

namespace pqt {

constexpr int kExactThreads = 256;
constexpr int kExactPer = PQT_MAX_K / kExactThreads;     // entries of the short list per thread
constexpr int kExactBits = 10, kExactBins = 1 << kExactBits;
constexpr int kExactBinMax = 64;                         // keys that may be ranked against their bin

template <typename Elem>
__global__ __launch_bounds__(kExactThreads) void exact_rerank_kernel(ExactArgs g) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int D = g.D, nd4 = D / 4, ks = g.k_short, k = g.k;
    float4* sy = reinterpret_cast<float4*>(smem);                                        // D floats
    unsigned long long* keys = reinterpret_cast<unsigned long long*>(smem + sizeof(float) * D);   // next_pow2(ks), >= 64
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int64_t q = blockIdx.x;
    const Elem* X = reinterpret_cast<const Elem*>(g.vectors);

    uint32_t* hist = reinterpret_cast<uint32_t*>(smem + sizeof(float) * D + sizeof(unsigned long long) * next_pow2(ks < 64 ? 64 : ks));
    uint32_t* part = hist + kExactBins;
    uint32_t* misc = part + kExactThreads / kWave;

    for (int c4 = tid; c4 < nd4; c4 += kExactThreads) sy[c4] = reinterpret_cast<const float4*>(g.queries + q * D)[c4];
    const int npad = next_pow2(ks) < 64 ? 64 : next_pow2(ks);
    // an entry without a vector (id -1) keeps a key that no vector has
    for (int e = tid; e < npad; e += kExactThreads) keys[e] = e < ks ? (unsigned long long)g.short_ids[q * ks + e] : ~0ull;
    for (int e = tid; e < kExactBins; e += kExactThreads) hist[e] = 0u;
    if (tid < 4) misc[tid] = tid == 0 ? 0xffffffffu : 0u;        // smallest and largest key, results' bin, a crowded bin
    __syncthreads();

    const int npieces = D / Piece<Elem>::kElems;                 // D is a multiple of the piece (checked by the caller)
    const int lpr = lanes_per_row(npieces);
    const int rows_per_wave = kWave / lpr, sub = lane / lpr, l = lane & (lpr - 1);
    const int rows_per_iter = rows_per_wave * (kExactThreads / kWave);
    const float* y = reinterpret_cast<const float*>(sy);
    constexpr int kRows = 4;
    uint32_t low = 0xffffffffu, high = 0u;
    for (int c0 = wave * rows_per_wave + sub; c0 < ks; c0 += kRows * rows_per_iter) {
        const Elem* x[kRows];
        bool have[kRows];
        float acc[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int c = c0 + u * rows_per_iter;
            const long long id = c < ks ? (long long)keys[c] : -1;
            have[u] = id >= 0;
            x[u] = have[u] ? X + (size_t)id * D : reinterpret_cast<const Elem*>(g.queries + q * D);   // (something that may be read)
            acc[u] = 0.0f;
        }
        for (int piece = l; piece < npieces; piece += lpr) {
            uint4 raw[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) raw[u] = reinterpret_cast<const uint4*>(x[u])[piece];
#pragma unroll
            for (int u = 0; u < kRows; ++u) acc[u] = Piece<Elem>::add(raw[u], piece, y, acc[u]);
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            for (int off = 1; off < lpr; off <<= 1) acc[u] += __shfl_xor(acc[u], off, kWave);
            const int c = c0 + u * rows_per_iter;
            if (have[u] && l == 0) {
                const uint32_t bits = mono_key(acc[u]);
                keys[c] = ((unsigned long long)bits << 32) | (uint32_t)keys[c];
                low = min(low, bits);
                high = max(high, bits);
            }
        }
    }
    low = wave_min_u32(low);
    high = wave_max_u32(high);
    if (lane == 0) {
        atomicMin(&misc[0], low);
        atomicMax(&misc[1], high);
    }
    __syncthreads();

    // ---- the k smallest ---------------------------------------------------------------------------------------
    const uint32_t lo_key = misc[0], range = misc[1] >= lo_key ? misc[1] - lo_key : 0u;
    const int width = 32 - __clz((int)(range | 1u)), shift = width > kExactBits ? width - kExactBits : 0;
    unsigned long long mine[kExactPer];
    auto bin_of = [&](unsigned long long key) { return ((uint32_t)(key >> 32) - lo_key) >> shift; };
#pragma unroll
    for (int u = 0; u < kExactPer; ++u) {
        const int e = tid + u * kExactThreads;
        mine[u] = e < ks ? keys[e] : ~0ull;
        if (mine[u] != ~0ull) atomicAdd(&hist[bin_of(mine[u])], 1u);
    }
    __syncthreads();
    constexpr int per = kExactBins / kExactThreads;
    uint32_t sum = 0, total;
#pragma unroll
    for (int j = 0; j < per; ++j) sum += hist[tid * per + j];
    uint32_t at = block_exclusive_sum(sum, part, total);
    const uint32_t kk = min((uint32_t)k, total);                 // results that exist
#pragma unroll
    for (int j = 0; j < per; ++j) {                              // counts -> first positions
        const uint32_t cnt = hist[tid * per + j];
        hist[tid * per + j] = at;
        if (at < kk && kk <= at + cnt) misc[2] = (uint32_t)(tid * per + j);
        if (at < kk && cnt > (uint32_t)kExactBinMax) misc[3] = 1u;
        at += cnt;
    }
    __syncthreads();
    if (misc[3] == 0u) {
        const uint32_t last = misc[2];
#pragma unroll
        for (int u = 0; u < kExactPer; ++u)
            if (mine[u] != ~0ull && bin_of(mine[u]) <= last) keys[atomicAdd(&hist[bin_of(mine[u])], 1u)] = mine[u];
        __syncthreads();                                         // hist[b] is now the end of bin b, the start of bin b + 1
#pragma unroll
        for (int u = 0; u < kExactPer; ++u) {
            if (mine[u] == ~0ull || bin_of(mine[u]) > last) continue;
            const uint32_t bin = bin_of(mine[u]), first = bin ? hist[bin - 1] : 0u, end = hist[bin];
            uint32_t r = first;
            for (uint32_t x = first; x < end; ++x) r += keys[x] < mine[u] ? 1u : 0u;
            if (r < kk) {
                g.out_ids[q * k + r] = (int64_t)(uint32_t)mine[u];
                g.out_dists[q * k + r] = mono_inv((uint32_t)(mine[u] >> 32));
            }
        }
        for (int e = (int)kk + tid; e < k; e += kExactThreads) {
            g.out_ids[q * k + e] = -1;
            g.out_dists[q * k + e] = __builtin_inff();
        }
        return;
    }
    block_sort_lds<4>(keys, npad, tid, kExactThreads);
    for (int e = tid; e < k; e += kExactThreads) {
        const unsigned long long key = keys[e];
        if (key == ~0ull) {
            g.out_ids[q * k + e] = -1;
            g.out_dists[q * k + e] = __builtin_inff();
        } else {
            g.out_ids[q * k + e] = (int64_t)(uint32_t)key;
            g.out_dists[q * k + e] = mono_inv((uint32_t)(key >> 32));
        }
    }
}

size_t exact_lds_bytes(int D, int k_short) {
    const int npad = next_pow2(k_short) < 64 ? 64 : next_pow2(k_short);
    return sizeof(float) * D + sizeof(unsigned long long) * npad + sizeof(uint32_t) * (kExactBins + kExactThreads / kWave + 4);
}

hipError_t launch_exact_rerank(const ExactArgs& a, hipStream_t s) {
    if (a.nq <= 0) return hipSuccess;
    const size_t lds = exact_lds_bytes(a.D, a.k_short);
    if (a.elem_bytes == 4)
        hipLaunchKernelGGL(exact_rerank_kernel<float>, dim3((unsigned)a.nq), dim3(kExactThreads), lds, s, a);
    else
        hipLaunchKernelGGL(exact_rerank_kernel<uint8_t>, dim3((unsigned)a.nq), dim3(kExactThreads), lds, s, a);
    return hipGetLastError();
}

}  // namespace pqt
