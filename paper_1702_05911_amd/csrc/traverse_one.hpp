// Tree traversal of one query by one workgroup, its results in LDS: the first part of the kernel that answers a query of a small
// batch (query_kernel in rerank_kernel.hpp).  The values are those of traverse_kernel to the bit: the same matrix instruction,
// of whose sixteen rows the query is the first, the same sums in the same order.
#pragma once
#include "pqt_device.hpp"
#include "pqt_kernels.hpp"

namespace pqt {

// (The query is read in 16-byte pieces.)
struct TraverseOneLds {
    size_t off_key, off_q, off_qn, off_d1, off_sel, total;
};
__host__ __device__ constexpr TraverseOneLds traverse_one_layout(int D, int P, int k1, int k2, int M, int w) {
    TraverseOneLds L = {};
    size_t o = 0;
    L.off_key = o; o += (sizeof(unsigned long long) * P * w * k2 + 15) & ~size_t(15);
    L.off_q = o;   o += sizeof(float) * ((D + 3) & ~3);
    L.off_qn = o;  o += sizeof(float) * M;
    L.off_d1 = o;  o += sizeof(float) * P * k1;
    L.off_sel = o; o += sizeof(int) * P * w;
    L.total = (o + 15) & ~size_t(15);
    return L;
}
static_assert(traverse_one_layout(96, 1, 16, 7, 8, 5).off_q % 16 == 0 && traverse_one_layout(96, 1, 16, 7, 8, 5).off_key % 8 == 0,
              "a list of odd length");
// lists of up to 256 entries from the interleaved codebook
inline bool traverse_one_possible(const TraverseArgs& a) { return a.C2t != nullptr && a.w * a.k2 <= 4 * kWave; }

// A list of at most 64 E keys, sorted, to sLd / sLid; by one wavefront.
template <int E>
__device__ __forceinline__ void sort_list(const unsigned long long* keys, int R, int lane, float* sLd, uint32_t* sLid) {
    unsigned long long key[E];
#pragma unroll
    for (int r = 0; r < E; ++r) key[r] = lane + r * kWave < R ? keys[lane + r * kWave] : ~0ull;
    wave_sort_chunk<E>(key, lane, 0u);
#pragma unroll
    for (int r = 0; r < E; ++r)
        if (lane + r * kWave < R) {
            sLd[lane + r * kWave] = mono_inv((uint32_t)(key[r] >> 32));
            sLid[lane + r * kWave] = (uint32_t)key[r];
        }
}

// Query q: level-1 distances to sa[M][k1], sorted lists to sLd, sLid[P][R].  tmp: the LDS that traverse_one_layout describes.
// meanwhile(first): what the threads from `first` on do while those before sort; sa is complete by then.
// All threads call it; ends with a barrier.
template <typename Meanwhile>
__device__ __forceinline__ void traverse_one(const TraverseArgs& g, int64_t q, unsigned char* tmp, float* sa, float* sLd, uint32_t* sLid,
                                             Meanwhile&& meanwhile) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const TraverseOneLds L = traverse_one_layout(g.D, g.P, g.k1, g.k2, g.M, g.w);
    float* sq = reinterpret_cast<float*>(tmp + L.off_q);
    float* sqn = reinterpret_cast<float*>(tmp + L.off_qn);
    float* sd1 = reinterpret_cast<float*>(tmp + L.off_d1);
    int* ssel = reinterpret_cast<int*>(tmp + L.off_sel);
    unsigned long long* skey = reinterpret_cast<unsigned long long*>(tmp + L.off_key);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), nt = blockDim.x, nwaves = nt / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int D = g.D, P = g.P, k1 = g.k1, k2 = g.k2, M = g.M, w = g.w;
    const int dp = D / P, ds = D / M, per = M / P, R = w * k2;

    for (int d = tid; d < D; d += nt) sq[d] = g.queries[q * D + d];
    __syncthreads();
    for (int m = tid; m < M; m += nt) {
        float s = 0.0f;
#pragma unroll 8
        for (int d = 0; d < ds; ++d) s = fmaf(sq[m * ds + d], sq[m * ds + d], s);
        sqn[m] = s;
    }
    // ---- level 1: one job = (sub-part, tile of 16 centroids) -----------------------------------
    const int ntiles = (k1 + 15) / 16, row = lane & 15, kq = lane >> 4;
    constexpr int kJobs = 2;                                 // their accumulators wait for the norms
    for (int j0 = wave; j0 < M * ntiles; j0 += kJobs * nwaves) {
        v4f acc[kJobs];
#pragma unroll
        for (int u = 0; u < kJobs; ++u) {
            acc[u] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
            const int job = j0 + u * nwaves;
            if (job >= M * ntiles) continue;                 // the same for the wavefront
            const int m = job / ntiles, p = m / per, lo = m * ds - p * dp, col = job % ntiles * 16 + row;
            const float* arow = sq + m * ds;
            const float* brow = g.C1 + ((size_t)p * k1 + (col < k1 ? col : 0)) * dp + lo;
            for (int k0 = 0; k0 < ds; k0 += 32) {
                float bv[8];
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const int kd = k0 + 4 * s + kq;
                    bv[s] = (kd < ds && col < k1) ? brow[kd] : 0.0f;
                }
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const int kd = k0 + 4 * s + kq;
                    if (k0 + 4 * s < ds)
                        acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(row == 0 && kd < ds ? arow[kd] : 0.0f, bv[s], acc[u], 0, 0, 0);
                }
            }
        }
        if (j0 == wave) __syncthreads();                     // the norms (every wavefront has a first round: see below)
#pragma unroll
        for (int u = 0; u < kJobs; ++u) {
            const int job = j0 + u * nwaves, col = job % ntiles * 16 + row, m = job / ntiles;
            if (job < M * ntiles && kq == 0 && col < k1) sa[m * k1 + col] = (sqn[m] + g.c1n[m * k1 + col]) - 2.0f * acc[u][0];
        }
    }
    if (wave >= M * ntiles) __syncthreads();                 // (no job: the barrier of the first round)
    __syncthreads();
    // ---- per-part distances and the w closest clusters -------------------------------------------
    for (int e = tid; e < P * k1; e += nt) {
        const int i = e % k1, p = e / k1;
        float s = sa[p * per * k1 + i];
        for (int m = p * per + 1; m < (p + 1) * per; ++m) s += sa[m * k1 + i];
        sd1[e] = s;
    }
    __syncthreads();
    for (int e = tid; e < P * k1; e += nt) {
        const int i = e % k1, p = e / k1;
        const float* own = sd1 + p * k1;
        const unsigned long long me = ((unsigned long long)mono_key(own[i]) << 32) | (unsigned)i;
        int rank = 0;
        for (int j = 0; j < k1; ++j) rank += (((unsigned long long)mono_key(own[j]) << 32) | (unsigned)j) < me ? 1 : 0;
        if (rank < w) ssel[p * w + rank] = i;
    }
    __syncthreads();
    // ---- level 2: a thread per child ---------------------------------------------------------------
    const int nd4 = dp / 4;
    for (int e = tid; e < P * R; e += nt) {
        const int p = e / R, s = (e - p * R) / k2, j = e - p * R - s * k2, i = ssel[p * w + s];
        const v4f* child = reinterpret_cast<const v4f*>(g.C2t) + ((size_t)p * k1 + i) * nd4 * k2 + j;
        const float4* y = reinterpret_cast<const float4*>(sq + p * dp);
        float acc = 0.0f;
        for (int d0 = 0; d0 < nd4; d0 += 16) {
            v4f c[16];                                       // asked for together (see level2_lists)
#pragma unroll
            for (int u = 0; u < 16; ++u) c[u] = child[(size_t)(d0 + u < nd4 ? d0 + u : nd4 - 1) * k2];
            asm volatile("" : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]), "+v"(c[4]), "+v"(c[5]), "+v"(c[6]), "+v"(c[7]),
                              "+v"(c[8]), "+v"(c[9]), "+v"(c[10]), "+v"(c[11]), "+v"(c[12]), "+v"(c[13]), "+v"(c[14]), "+v"(c[15]));
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                if (d0 + u >= nd4) break;
                const float4 v = y[d0 + u];
                float diff = v.x - c[u][0];
                acc = fmaf(diff, diff, acc);
                diff = v.y - c[u][1];
                acc = fmaf(diff, diff, acc);
                diff = v.z - c[u][2];
                acc = fmaf(diff, diff, acc);
                diff = v.w - c[u][3];
                acc = fmaf(diff, diff, acc);
            }
        }
        skey[e] = ((unsigned long long)mono_key(acc) << 32) | (uint32_t)(i * k2 + j);
    }
    __syncthreads();
    if (wave < P) {                                          // (at most four parts)
        const int p = wave;
        if (R <= kWave) sort_list<1>(skey + p * R, R, lane, sLd + p * R, sLid + p * R);
        else if (R <= 2 * kWave) sort_list<2>(skey + p * R, R, lane, sLd + p * R, sLid + p * R);
        else sort_list<4>(skey + p * R, R, lane, sLd + p * R, sLid + p * R);
    } else {
        meanwhile(P * kWave);
    }
    if (P * kWave >= nt) meanwhile(0);                       // (four parts, 256 threads: nobody was left)
    __syncthreads();
}

}  // namespace pqt
