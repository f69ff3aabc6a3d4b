// The offline phase's per-vector work (Sec. 3.1 "bin map", Sec. 3.3 "Offline computation"): every database vector is put into
// its bin (nearest level-1 cluster of every tree part, nearest child of that cluster) and gets its line-quantisation code;
// every training vector votes for its nearest lines.  All of it starts from the level-1 sub-part distances of Sec. 3.3's last
// paragraph, so one kernel does it, and the distances never leave the chip.
//
// One workgroup per 64 vectors.  A wavefront takes a sub-part: the [64 x ds] . [ds x k1] products on the matrix cores (the
// traversal's instruction, order and rounding, so a vector falls into the bin the query path looks for it in), distances to
// LDS with the vector fastest; then a lane owns a vector and walks the code points (or lines), which are the same for
// the wavefront and come through the scalar cache, and nothing is compared across lanes.  Sub-part distances are added to
// the part's in ascending order; level 2 spreads (vector, child) pairs over the lanes, children of a cluster interleaved.
//
// Bound by vector instructions (six per vector, sub-part and code point) and, above 32 centroids, LDS reads (two of them): up to 32 the code search
// has a lane's distances in registers (2,000,003 vectors, below: the whole call 2.73 -> 2.29 ms). 2,000,003 vectors x 128, P = 2, k1 = 16, k2 = 8,
// M = 8, table codes: 1.62 ms (code search 0.62, level 2 0.3); the traversal kernel with w = 1 (one wavefront per list, 8 of 64 lanes at work), its
// distances written and read back, and one wavefront per vector for the codes took 7.0.  With staged values and distances side by side in LDS three
// workgroups instead of five fit a compute unit: 2.9.
#include <type_traits>

#include "pqt_device.hpp"
#include "pqt_kernels.hpp"

namespace pqt {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) uint32_t* scalar_words;

constexpr int kPlaceRows = kWave;              // vectors of a workgroup: one per lane
constexpr int kRowStride = kPlaceRows + 1;     // of a centroid's distances
constexpr int kSlab = 32;                      // dimensions of a sub-part staged at a time

struct PlaceLds {
    int st;                                    // row stride of a staged slab (floats): an odd number of 16-byte pieces
    size_t a_stride;                           // of a wavefront's distances (floats)
    size_t off_x, off_a, off_d1, off_sel, off_leaf, off_code, total;
};

__host__ __device__ constexpr PlaceLds place_layout(int ds, int P, int k1, int code_bytes, int waves, bool votes) {
    PlaceLds L = {};
    const int pieces = ((ds < kSlab ? ds : kSlab) + 3) / 4;
    L.st = 4 * (pieces | 1);
    size_t o = 0;
    L.off_x = o;    o += sizeof(float) * waves * kPlaceRows * L.st;
    // the distances of up to 32 centroids come out of one pass over the staged values and take their place
    const size_t x_bytes = sizeof(float) * kPlaceRows * L.st, a_bytes = sizeof(float) * k1 * kRowStride;
    // (whole 16-byte pieces: every wavefront's staged values are written in them)
    L.a_stride = ((k1 <= 32 && x_bytes > a_bytes ? x_bytes : a_bytes) + 15) / 16 * 4;
    if (k1 <= 32) o = 0;
    L.off_a = o;    o += sizeof(float) * waves * L.a_stride;
    L.off_d1 = o;   o += votes ? 0 : sizeof(float) * k1 * kRowStride;
    o = (o + 7) & ~size_t(7);
    L.off_sel = o;  o += votes ? 0 : sizeof(unsigned long long) * P * kPlaceRows;
    L.off_leaf = o; o += votes ? 0 : sizeof(unsigned long long) * P * kPlaceRows;
    L.off_code = o; o += votes ? 0 : (size_t)kPlaceRows * code_bytes;
    L.total = (o + 15) & ~size_t(15);
    return L;
}

// Where a wavefront stages its values
__host__ __device__ constexpr size_t staging_stride(const PlaceLds& L, int k1) {
    return k1 <= 32 ? L.a_stride : (size_t)kPlaceRows * L.st;
}
constexpr bool staging_is_aligned() {
    for (int ds = 4; ds <= 36; ds += 4)
        for (int k1 = 1; k1 <= 40; ++k1) {
            const PlaceLds L = place_layout(ds, 2, k1, 4, 4, false);
            if (L.off_x % 16 || L.st % 4 || staging_stride(L, k1) % 4) return false;
        }
    return true;
}
static_assert(staging_is_aligned(), "16-byte writes");

// Level-1 distances of the workgroup's vectors in sub-part m: at[i * kRowStride + v].  By one wavefront, or (SHARED) by all of
// the workgroup, which stage the values together and take two tiles of 16 centroids each in turn.
// WIDE: rows are read in 16-byte pieces.  ROWS: vectors, 64 or 16 (at: ROWS + 1 values a centroid).  Vectors past the end
// repeat the last one.
template <bool WIDE, bool SHARED = false, int ROWS = kPlaceRows>
__device__ __forceinline__ void subpart_distances(const PlaceArgs& g, int64_t v0, int nv, int m, int st, float* xs, float* at) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = SHARED ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave) : 0, waves = SHARED ? (int)blockDim.x / kWave : 1;
    auto ordered = [&]() {
        if (SHARED) __syncthreads(); else wave_lds_order();
    };
    const int k1 = g.k1, dp = g.D / g.P, ds = g.D / g.M, per = g.M / g.P;
    const int p = m / per, lo = m * ds - p * dp;
    const int ntiles = (k1 + 15) / 16, row = lane & 15, kq = lane >> 4;
    const float* x = g.x + (size_t)v0 * g.D + (size_t)m * ds;
    constexpr int kTiles = ROWS / 16;
    float norm = 0.0f;                                       // of vector `lane` (mod ROWS)
    for (int nt0 = 0; nt0 < ntiles; nt0 += 2 * waves) {
        const int nt = nt0 + 2 * wave;
        const bool one = !SHARED || nt < ntiles;
        const bool two = nt + 1 < ntiles;                    // two tiles of 16 centroids per pass over the values
        v4f acc[2][kTiles];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < kTiles; ++r) acc[t][r] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        for (int k0 = 0; k0 < ds; k0 += kSlab) {
            const int width = ds - k0 < kSlab ? ds - k0 : kSlab;
            if (nt0 == 0 || ds > kSlab) {
                ordered();
                if (WIDE) {
                    const int pieces = width / 4;
                    int shift = 0;
                    while ((1 << shift) < pieces) ++shift;
                    const int c = min(lane & ((1 << shift) - 1), pieces - 1), step = (kWave >> shift) * waves;
                    const int r0 = (lane >> shift) + (kWave >> shift) * wave;
#pragma unroll 4
                    for (int r = r0; r < ROWS; r += step)
                        *reinterpret_cast<float4*>(xs + r * st + 4 * c) =
                            *reinterpret_cast<const float4*>(x + (size_t)min(r, nv - 1) * g.D + k0 + 4 * c);
                } else {
                    const int c = lane & (kSlab - 1);
                    if (c < ((width + 3) & ~3))
                        for (int r = lane / kSlab + kWave / kSlab * wave; r < ROWS; r += kWave / kSlab * waves)
                            xs[r * st + c] = c < width ? x[(size_t)min(r, nv - 1) * g.D + k0 + c] : 0.0f;
                }
                ordered();
                if (nt0 == 0)
                    for (int d = 0; d < width; ++d) norm = fmaf(xs[lane % ROWS * st + d], xs[lane % ROWS * st + d], norm);
            }
            if (!one) continue;
            // the centroid values of eight steps are fetched together, so that their latencies overlap
            float bv[2][8];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int col = (nt + t) * 16 + row;
                const float* brow = g.C1 + ((size_t)p * k1 + (col < k1 ? col : 0)) * dp + lo;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int kd = k0 + 4 * u + kq;
                    bv[t][u] = (t == 0 || two) && kd < ds && col < k1 ? brow[kd] : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (4 * u < width) {                         // uniform
#pragma unroll
                    for (int r = 0; r < kTiles; ++r) {
                        const float av = xs[(r * 16 + row) * st + 4 * u + kq];
                        acc[0][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[0][u], acc[0][r], 0, 0, 0);
                        if (two) acc[1][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[1][u], acc[1][r], 0, 0, 0);
                    }
                }
            }
        }
        if (!SHARED) wave_lds_order();                       // (the distances may take the staged values' place)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (!one) break;
            const int col = (nt + t) * 16 + row;
            const float cn = g.c1n[m * k1 + (col < k1 ? col : 0)];
#pragma unroll
            for (int r = 0; r < kTiles; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int v = r * 16 + 4 * kq + j;
                    const float xn = __shfl(norm, v, kWave);
                    if (col < k1 && (t == 0 || two)) at[col * (ROWS + 1) + v] = (xn + cn) - 2.0f * acc[t][r][j];
                }
        }
    }
    ordered();
}

// The nearest of the 256 code points of a sub-part: the smallest (Eq. 9 value, number).  Eight values at a time only
// their minimum is compared; the eight that hold the smallest are looked at again.  K > 0: the distances of up to K centroids stay in
// registers, which the code points' centroid numbers, the same for the wavefront, index; 0: they are read from LDS.
template <int K>
__device__ __forceinline__ uint32_t nearest_code(const CodeEntry* table, const float* at, int k1) {
    typedef float Distances __attribute__((ext_vector_type(K > 0 ? K : 1)));
    const int lane = threadIdx.x & (kWave - 1);
    scalar_words w = (scalar_words)(uintptr_t)table;
    auto value = [&](uint32_t ij, float lam, float kc) {
        const float b2 = at[(ij & 0xffu) * kRowStride + lane], a2 = at[((ij >> 8) & 0xffu) * kRowStride + lane];
        return fmaf(lam, a2 - b2, b2) + kc;
    };
    Distances d;
    if constexpr (K > 0) {
#pragma unroll
        for (int i = 0; i < K; ++i) d[i] = at[min(i, k1 - 1) * kRowStride + lane];
    }
    auto scalar_value = [&](uint32_t ij, float lam, float kc) {
        if constexpr (K > 0) {
            const float b2 = d[ij & (K - 1)], a2 = d[(ij >> 8) & (K - 1)];
            return fmaf(lam, a2 - b2, b2) + kc;
        } else {
            return value(ij, lam, kc);
        }
    };
    float best = __builtin_inff();
    int block = 0;
    for (int c = 0; c < 256; c += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = scalar_value(w[3 * (c + u)], __uint_as_float(w[3 * (c + u) + 1]), __uint_as_float(w[3 * (c + u) + 2]));
        const float low = fminf(fminf(fminf(v[0], v[1]), fminf(v[2], v[3])), fminf(fminf(v[4], v[5]), fminf(v[6], v[7])));
        if (low < best) {
            best = low;
            block = c;
        }
    }
    uint32_t code = (uint32_t)block;
#pragma unroll
    for (int u = 7; u >= 0; --u) {
        const CodeEntry e = table[block + u];
        if (value(e.ij, e.lam, e.kc) == best) code = (uint32_t)(block + u);
    }
    if (__any(!(best < __builtin_inff()))) {                 // no finite value: by the order of the keys, as everywhere
        uint32_t low = 0xffffffffu, first = 0u;
        for (int c = 0; c < 256; ++c) {
            const uint32_t key = mono_key(value(w[3 * c], __uint_as_float(w[3 * c + 1]), __uint_as_float(w[3 * c + 2])));
            if (key < low || c == 0) {
                low = key;
                first = (uint32_t)c;
            }
        }
        if (!(best < __builtin_inff())) code = first;
    }
    return code;
}

// (pair, lambda) codes (Sec. 3.3 "Offline computation"; Eq. 7 stored directly).  A code stands for the
// point (1 - lambda) c_i + lambda c_j with lambda = (level - 96) / 16; a sub-vector gets the code of
// the nearest such point.  With b^2, a^2 its own distances to c_i, c_j and c^2 = ||c_i - c_j||^2, the projection on the line
// is at (b^2 - a^2 + c^2) / (2 c^2); the level nearest to it (clamped to a byte) is the line's nearest
// code point, whose distance is Eq. 9 on the same values.  The smallest (distance, pair number) wins;
// pairs with c^2 = 0 never do.  `table` holds the pairs (entry = pair number, kc = c^2).
__device__ __forceinline__ uint32_t nearest_pair(const CodeEntry* table, int npairs, const float* at) {
    const int lane = threadIdx.x & (kWave - 1);
    scalar_words w = (scalar_words)(uintptr_t)table;
    uint32_t low = 0xffffffffu;
    int best = -1;
    uint32_t best_level = 96;                                // no usable pair: pair 0 at lambda = 0
    for (int c = 0; c < npairs; ++c) {
        const uint32_t ij = w[3 * c];
        const float kc = __uint_as_float(w[3 * c + 2]);
        if (!(kc > 0.0f)) continue;                          // the same for the wavefront
        const float b2 = at[(ij & 0xffu) * kRowStride + lane], a2 = at[((ij >> 8) & 0xffu) * kRowStride + lane];
        const float proj = ((b2 - a2) + kc) / (2.0f * kc);
        const float level = fminf(fmaxf(floorf(fmaf(proj, 16.0f, 96.5f)), 0.0f), 255.0f);
        const float lam = fmaf(level, 0.0625f, -6.0f);
        const uint32_t key = mono_key(fmaf(fmaf(lam, lam, -lam), kc, fmaf(lam, a2 - b2, b2)));
        if (key < low || best < 0) {
            low = key;
            best = c;
            best_level = (uint32_t)level;
        }
    }
    return (uint32_t)(best < 0 ? 0 : best) | (best_level << 8);
}

// The nearest line of a training sub-vector (Sec. 3.3 "Offline computation") among the pairs c0 .. c1 - 1.  With b^2, a^2 its
// level-1 distances to c_i, c_j and c^2 = ||c_i - c_j||^2: the projection lies at lambda = (b^2 - a^2 + c^2) / (2 c^2) and
// misses the vector by b^2 - lambda^2 c^2.  Returns the smallest (ordered bits of the error) << 32 | pair number; pairs of
// coinciding centroids never win, ~0 when there are no others.  Eight pairs at a time, so that their latencies overlap.
__device__ __forceinline__ float line_lambda(float b2, float a2, float c2) { return ((b2 - a2) + c2) / (2.0f * c2); }

__device__ __forceinline__ unsigned long long nearest_line(const LinePair* pairs, int c0, int c1, const float* at) {
    const int lane = threadIdx.x & (kWave - 1);
    scalar_words w = (scalar_words)(uintptr_t)pairs;
    uint32_t low = 0xffffffffu;
    int best = -1;
    constexpr int kBlock = 8;
    auto look_at = [&](int c, auto whole) {
        uint32_t ij[kBlock], key[kBlock];
        float c2[kBlock], b2[kBlock], a2[kBlock];
#pragma unroll
        for (int u = 0; u < kBlock; ++u) {
            const int p = decltype(whole)::value ? c + u : min(c + u, c1 - 1);      // (past the end: the last pair again)
            ij[u] = w[2 * p];
            c2[u] = __uint_as_float(w[2 * p + 1]);
        }
#pragma unroll
        for (int u = 0; u < kBlock; ++u) {
            b2[u] = at[(ij[u] & 0xffffu) * kRowStride + lane];
            a2[u] = at[(ij[u] >> 16) * kRowStride + lane];
        }
#pragma unroll
        for (int u = 0; u < kBlock; ++u) {
            const float lam = line_lambda(b2[u], a2[u], c2[u]);
            key[u] = mono_key(fmaf(-lam * lam, c2[u], b2[u]));
        }
#pragma unroll
        for (int u = 0; u < kBlock; ++u) {
            if (!(c2[u] > 0.0f)) continue;                   // the same for the wavefront
            if (key[u] < low || best < 0) {                  // (the last pair again: equal to itself)
                low = key[u];
                best = c + u;
            }
        }
    };
    int c = c0;
    for (; c + kBlock <= c1; c += kBlock) look_at(c, std::true_type{});
    if (c < c1) look_at(c, std::false_type{});
    return best < 0 ? ~0ull : ((unsigned long long)low << 32) | (uint32_t)best;
}

// The vote: sub-part << 48 | pair number << 32 | ordered bits of lambda; pair number 0xffff when the sub-part has no usable pair.
__device__ __forceinline__ unsigned long long vote_of(const LinePair* pairs, unsigned long long nearest, int m, const float* at) {
    const int lane = threadIdx.x & (kWave - 1);
    if (nearest == ~0ull) return ((unsigned long long)m << 48) | 0xffffffffffffull;
    const uint32_t p = (uint32_t)nearest;
    const LinePair pr = pairs[p];
    const float lam = line_lambda(at[(pr.ij & 0xffffu) * kRowStride + lane], at[(pr.ij >> 16) * kRowStride + lane], pr.c2);
    return ((unsigned long long)m << 48) | ((unsigned long long)p << 32) | mono_key(lam);
}

enum { kTableCodes, kPairCodes, kVotes };

// What place_kernel ends with, for ROWS vectors, by the whole workgroup: sel[p * ROWS + v] holds the nearest cluster of every part, code the codes
// of cb bytes; leaf[] starts as all ones.  (place_kernel has it inline: called from there it was scheduled so that 60,000 vectors x 960 took 690 us
// instead of 515.)  A lane per (vector, child) at level 2, as 16 vectors are few: with four lanes a vector (nearest_child), the parts side by side,
// up to eight children would gain (1,000 x 960, four parts of eight 65 -> 43 us, x 128, two parts 27 -> 25), 32 lose (x 96 28 -> 38).
template <int ROWS, bool WIDE>
__device__ __forceinline__ void finish_vectors(const PlaceArgs& g, int64_t v0, int nv, const unsigned long long* sel, unsigned long long* leaf,
                                               const uint8_t* code, int cb) {
    const int tid = threadIdx.x, nt = blockDim.x, D = g.D, P = g.P, k1 = g.k1, k2 = g.k2, dp = D / P;
    // ---- level 2: the children of the nearest cluster, plain squared differences, dimensions in ascending order ----
    const int nd4 = dp / 4;
    for (int p = 0; p < P; ++p)
        for (int e = tid; e < ROWS * k2; e += nt) {
            const int v = e / k2, j = e - v * k2;
            if (v >= nv) continue;
            const uint32_t i = (uint32_t)sel[p * ROWS + v];
            const float* y = g.x + (size_t)(v0 + v) * D + (size_t)p * dp;
            float acc = 0.0f;
            if (WIDE && g.C2t) {
                const float4* c = reinterpret_cast<const float4*>(g.C2t) + ((size_t)p * k1 + i) * nd4 * k2 + j;
#pragma unroll 4
                for (int d = 0; d < nd4; ++d) {
                    const float4 yv = *reinterpret_cast<const float4*>(y + 4 * d), cv = c[(size_t)d * k2];
                    float diff = yv.x - cv.x;
                    acc = fmaf(diff, diff, acc);
                    diff = yv.y - cv.y;
                    acc = fmaf(diff, diff, acc);
                    diff = yv.z - cv.z;
                    acc = fmaf(diff, diff, acc);
                    diff = yv.w - cv.w;
                    acc = fmaf(diff, diff, acc);
                }
            } else {
                const float* c = g.C2 + (((size_t)p * k1 + i) * k2 + j) * dp;
                for (int d = 0; d < dp; ++d) {
                    const float diff = y[d] - c[d];
                    acc = fmaf(diff, diff, acc);
                }
            }
            atomicMin(&leaf[p * ROWS + v], ((unsigned long long)mono_key(acc) << 32) | (i * (uint32_t)k2 + (uint32_t)j));
        }
    __syncthreads();
    if (tid < nv) {
        unsigned long long lin = 0;
        for (int p = 0; p < P; ++p) lin = lin * g.k1k2 + (uint32_t)leaf[p * ROWS + tid];
        g.slots[v0 + tid] = (uint32_t)(lin % g.H);
    }
    const int bytes = nv * cb;
    uint8_t* out = g.codes + (size_t)v0 * cb;
    if (((uintptr_t)out & 3u) == 0 && bytes % 4 == 0)
        for (int e = tid; e < bytes / 4; e += nt) reinterpret_cast<uint32_t*>(out)[e] = reinterpret_cast<const uint32_t*>(code)[e];
    else
        for (int e = tid; e < bytes; e += nt) out[e] = code[e];
}

// The nearest child of cluster i of part p for one vector: (ordered bits of the distance) << 32 | leaf, plain squared differences,
// dimensions in ascending order.  Four lanes share the vector: each brings every fourth 16 bytes of it, which the others take from its
// register in the subtraction itself, and works on every fourth child, two at a time.  What bounds it is the 64 bytes a clock that the
// vector cache returns: 9 loads per 16 dimensions and 128 (vector, child) pairs, 16 with a lane per pair that brings the vector for
// itself (2,000,003 vectors x 128, P = 2, k2 = 8: the kernel 1.74 -> 1.62 ms; 1,000,000 vectors, a call with one child 840 -> 797 us, two 868 and
// 784, four 845 and 786, 16 1,098 and 900, 32 1,813 and 1,061).
template <int U>
__device__ __forceinline__ float quad_value(float x) {       // of lane U of every four
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), U * 0x55, 0xf, 0xf, true));
}
template <int U>
__device__ __forceinline__ void child_step(const float4& y, const float4& c, float& acc) {
    float diff = quad_value<U>(y.x) - c.x;
    acc = fmaf(diff, diff, acc);
    diff = quad_value<U>(y.y) - c.y;
    acc = fmaf(diff, diff, acc);
    diff = quad_value<U>(y.z) - c.z;
    acc = fmaf(diff, diff, acc);
    diff = quad_value<U>(y.w) - c.w;
    acc = fmaf(diff, diff, acc);
}
__device__ __forceinline__ unsigned long long nearest_child(const PlaceArgs& g, int64_t v, int p, uint32_t i) {
    const int l = threadIdx.x & 3, k2 = g.k2, dp = g.D / g.P, nd4 = dp / 4;
    const float4* y = reinterpret_cast<const float4*>(g.x + (size_t)v * g.D + (size_t)p * dp);
    const float4* cluster = reinterpret_cast<const float4*>(g.C2t) + ((size_t)p * g.k1 + i) * nd4 * k2;
    unsigned long long best = ~0ull;
    for (int j0 = 0; j0 < k2; j0 += 8) {
        const int j = j0 + l;
        const bool two = j0 + 4 < k2;                        // the same for all lanes
        const float4* a = cluster + min(j, k2 - 1);
        const float4* b = cluster + min(j + 4, k2 - 1);
        float acc[2] = {0.0f, 0.0f};
        int d = 0;
        for (; d + 4 <= nd4; d += 4) {
            const float4 yv = y[d + l];
            float4 c[2][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) c[0][u] = a[(size_t)(d + u) * k2];
            if (two)
#pragma unroll
                for (int u = 0; u < 4; ++u) c[1][u] = b[(size_t)(d + u) * k2];
            child_step<0>(yv, c[0][0], acc[0]);
            child_step<1>(yv, c[0][1], acc[0]);
            child_step<2>(yv, c[0][2], acc[0]);
            child_step<3>(yv, c[0][3], acc[0]);
            if (two) {
                child_step<0>(yv, c[1][0], acc[1]);
                child_step<1>(yv, c[1][1], acc[1]);
                child_step<2>(yv, c[1][2], acc[1]);
                child_step<3>(yv, c[1][3], acc[1]);
            }
        }
        for (; d < nd4; ++d) {
            const float4 yv = y[d];                          // (the same in all four)
            child_step<0>(yv, a[(size_t)d * k2], acc[0]);
            if (two) child_step<0>(yv, b[(size_t)d * k2], acc[1]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const unsigned long long key = ((unsigned long long)mono_key(acc[u]) << 32) | (i * (uint32_t)k2 + (uint32_t)(j + 4 * u));
            if (j + 4 * u < k2 && key < best) best = key;
        }
    }
#pragma unroll
    for (int off = 1; off < 4; off <<= 1) {
        const unsigned long long o = __shfl_xor(best, off, kWave);
        best = o < best ? o : best;
    }
    return best;
}

// K: centroids whose distances the search for table codes has in registers (nearest_code).
template <int MODE, bool WIDE, int K>
__global__ __launch_bounds__(256, 5) void place_kernel(PlaceArgs g, PlaceLds L) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), nt = blockDim.x, waves = nt / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int D = g.D, P = g.P, k1 = g.k1, k2 = g.k2, M = g.M, dp = D / P, per = M / P;
    const int64_t v0 = (int64_t)blockIdx.x * kPlaceRows;
    const int nv = (int)(g.n - v0 < kPlaceRows ? g.n - v0 : kPlaceRows);
    float* xs = reinterpret_cast<float*>(smem + L.off_x) + wave * staging_stride(L, k1);
    float* a0 = reinterpret_cast<float*>(smem + L.off_a);
    float* d1 = reinterpret_cast<float*>(smem + L.off_d1);
    unsigned long long* sel = reinterpret_cast<unsigned long long*>(smem + L.off_sel);
    unsigned long long* leaf = reinterpret_cast<unsigned long long*>(smem + L.off_leaf);
    uint8_t* code = smem + L.off_code;
    float* at = a0 + (size_t)wave * L.a_stride;
    if (MODE != kVotes)
        for (int e = tid; e < P * kPlaceRows; e += nt) sel[e] = leaf[e] = ~0ull;

    for (int m0 = 0; m0 < M; m0 += waves) {
        const int m = m0 + wave;
        if (m < M) {
            subpart_distances<WIDE>(g, v0, nv, m, L.st, xs, at);
            if (MODE == kVotes) {
                const LinePair* pairs = g.pairs + (size_t)m * g.npairs;
                const unsigned long long vote = vote_of(pairs, nearest_line(pairs, 0, g.npairs, at), m, at);
                if (lane < nv) g.keys[(size_t)m * g.n + v0 + lane] = vote;
            } else if (MODE == kTableCodes) {
                code[lane * M + m] = (uint8_t)nearest_code<K>(g.table + (size_t)m * 256, at, k1);
            } else {
                const uint32_t c = nearest_pair(g.table + (size_t)m * 256, g.npairs, at);
                code[(lane * M + m) * 2] = (uint8_t)c;
                code[(lane * M + m) * 2 + 1] = (uint8_t)(c >> 8);
            }
        }
        if (MODE == kVotes) continue;
        __syncthreads();
        // the parts' distances: sub-parts in ascending order; a wavefront has its own centroids throughout
        for (int s = 0; s < waves && m0 + s < M; ++s) {
            const int q = (m0 + s) % per;
            const float* as = a0 + (size_t)s * L.a_stride + lane;
            unsigned long long best = ~0ull;
            for (int i = wave; i < k1; i += waves) {
                float sum = as[i * kRowStride];
                if (q > 0) sum += d1[i * kRowStride + lane];
                d1[i * kRowStride + lane] = sum;
                const unsigned long long key = ((unsigned long long)mono_key(sum) << 32) | (unsigned)i;
                best = key < best ? key : best;
            }
            if (q == per - 1) atomicMin(&sel[(m0 + s) / per * kPlaceRows + lane], best);
        }
        __syncthreads();
    }
    if (MODE == kVotes) return;

    // ---- level 2: the children of the nearest cluster, plain squared differences, dimensions in ascending order ----
    if (WIDE && g.C2t) {
        for (int p = 0; p < P; ++p)
            for (int v = tid / 4; v < kPlaceRows; v += nt / 4) {
                const unsigned long long key = nearest_child(g, v0 + min(v, nv - 1), p, (uint32_t)sel[p * kPlaceRows + v]);
                if ((tid & 3) == 0 && v < nv) leaf[p * kPlaceRows + v] = key;
            }
    } else {
        for (int p = 0; p < P; ++p)
            for (int e = tid; e < kPlaceRows * k2; e += nt) {
                const int v = e / k2, j = e - v * k2;
                if (v >= nv) continue;
                const uint32_t i = (uint32_t)sel[p * kPlaceRows + v];
                const float* y = g.x + (size_t)(v0 + v) * D + (size_t)p * dp;
                const float* c = g.C2 + (((size_t)p * k1 + i) * k2 + j) * dp;
                float acc = 0.0f;
                for (int d = 0; d < dp; ++d) {
                    const float diff = y[d] - c[d];
                    acc = fmaf(diff, diff, acc);
                }
                atomicMin(&leaf[p * kPlaceRows + v], ((unsigned long long)mono_key(acc) << 32) | (i * (uint32_t)k2 + (uint32_t)j));
            }
    }
    __syncthreads();
    if (tid < nv) {
        unsigned long long lin = 0;
        for (int p = 0; p < P; ++p) lin = lin * g.k1k2 + (uint32_t)leaf[p * kPlaceRows + tid];
        g.slots[v0 + tid] = (uint32_t)(lin % g.H);
    }
    const int cb = M * (MODE == kPairCodes ? 2 : 1), bytes = nv * cb;
    uint8_t* out = g.codes + (size_t)v0 * cb;
    if (((uintptr_t)out & 3u) == 0 && bytes % 4 == 0)
        for (int e = tid; e < bytes / 4; e += nt) reinterpret_cast<uint32_t*>(out)[e] = reinterpret_cast<const uint32_t*>(code)[e];
    else
        for (int e = tid; e < bytes; e += nt) out[e] = code[e];
}

// Few vectors: 16 per workgroup instead of 64, all sub-parts' distances at once, and a wavefront takes one vector's sub-part with
// the code points side by side in its lanes, as lone wavefronts that walk 256 code points take 20 us for a sub-part.  The same
// values, the smallest (value, number) wins as above.  Up to two workgroups per compute unit: x 128, P = 2, k1 = 16, M = 8,
// us per call, 64 vectors a workgroup and 16: 1,000 vectors 52 and 16, 8,192 57 and 34, 12,000 60 and 49 (M = 4: 39 and 41; D = 960,
// P = 4: 204 and 142).
constexpr int kFewRows = 16, kFewThreads = 1024, kFewVectors = 8192;
struct FewLds {
    int st;
    size_t off_x, off_sel, off_leaf, off_code, total;        // the distances come first: M x k1 x 17
};
__host__ __device__ constexpr FewLds few_layout(int ds, int P, int k1, int M, int code_bytes) {
    FewLds L = {};
    L.st = place_layout(ds, P, k1, code_bytes, 1, false).st;
    size_t o = (sizeof(float) * M * k1 * (kFewRows + 1) + 15) & ~size_t(15);
    L.off_x = o;    o += sizeof(float) * (kFewThreads / kWave) * kFewRows * L.st;
    L.off_sel = o;  o += sizeof(unsigned long long) * P * kFewRows;
    L.off_leaf = o; o += sizeof(unsigned long long) * P * kFewRows;
    L.off_code = o; o += (size_t)kFewRows * code_bytes;
    L.total = (o + 15) & ~size_t(15);
    return L;
}

__device__ __forceinline__ unsigned long long wave_min_key(unsigned long long v) {
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), off, kWave), lo = (uint32_t)__shfl_xor((int)(uint32_t)v, off, kWave);
        const unsigned long long o = ((unsigned long long)hi << 32) | lo;
        v = o < v ? o : v;
    }
    return v;
}

template <int MODE, bool WIDE>
__global__ __launch_bounds__(kFewThreads) void place_few_kernel(PlaceArgs g, FewLds L) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), waves = kFewThreads / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int P = g.P, k1 = g.k1, M = g.M, per = M / P;
    const int64_t v0 = (int64_t)blockIdx.x * kFewRows;
    const int nv = (int)(g.n - v0 < kFewRows ? g.n - v0 : kFewRows);
    float* a = reinterpret_cast<float*>(smem);
    float* xs = reinterpret_cast<float*>(smem + L.off_x) + (size_t)wave * kFewRows * L.st;
    unsigned long long* sel = reinterpret_cast<unsigned long long*>(smem + L.off_sel);
    unsigned long long* leaf = reinterpret_cast<unsigned long long*>(smem + L.off_leaf);
    uint8_t* code = smem + L.off_code;
    constexpr int kStride = kFewRows + 1;
    if (tid < P * kFewRows) sel[tid] = leaf[tid] = ~0ull;
    for (int m = wave; m < M; m += waves) subpart_distances<WIDE, false, kFewRows>(g, v0, nv, m, L.st, xs, a + (size_t)m * k1 * kStride);
    __syncthreads();
    // the parts' distances: sub-parts in ascending order
    for (int e = tid; e < P * k1 * kFewRows; e += kFewThreads) {
        const int v = e % kFewRows, i = e / kFewRows % k1, p = e / kFewRows / k1;
        const float* d = a + ((size_t)p * per * k1 + i) * kStride + v;
        float sum = d[0];
        for (int s = 1; s < per; ++s) sum = d[(size_t)s * k1 * kStride] + sum;
        atomicMin(&sel[p * kFewRows + v], ((unsigned long long)mono_key(sum) << 32) | (unsigned)i);
    }
    // codes: the entries of four units are fetched together
    constexpr int kUnits = 4;
    for (int u0 = wave; u0 < M * nv; u0 += kUnits * waves) {
        CodeEntry entry[kUnits][4];
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            const int m = min(u0 + u * waves, M * nv - 1) % M;
#pragma unroll
            for (int q = 0; q < 4; ++q) entry[u][q] = g.table[(size_t)m * 256 + q * kWave + lane];
        }
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            const int unit = u0 + u * waves, m = unit % M, v = unit / M;
            if (unit >= M * nv) break;                       // the same for the wavefront
            const float* at = a + (size_t)m * k1 * kStride + v;
            unsigned long long best = ~0ull;
            uint32_t best_level = 96;                        // no usable pair: pair 0 at lambda = 0
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const CodeEntry& e = entry[u][q];
                const int c = q * kWave + lane;
                if (MODE == kPairCodes && (c >= g.npairs || !(e.kc > 0.0f))) continue;
                const float b2 = at[(e.ij & 0xffu) * kStride], a2 = at[((e.ij >> 8) & 0xffu) * kStride];
                if (MODE == kTableCodes) {
                    const float value = fmaf(e.lam, a2 - b2, b2) + e.kc;
                    const unsigned long long key = ((unsigned long long)mono_key(value + 0.0f) << 32) | (unsigned)c;     // (no negative zero)
                    best = key < best ? key : best;
                } else {
                    const float proj = ((b2 - a2) + e.kc) / (2.0f * e.kc);
                    const float level = fminf(fmaxf(floorf(fmaf(proj, 16.0f, 96.5f)), 0.0f), 255.0f);
                    const float lam = fmaf(level, 0.0625f, -6.0f);
                    const uint32_t bits = mono_key(fmaf(fmaf(lam, lam, -lam), e.kc, fmaf(lam, a2 - b2, b2)));
                    const unsigned long long key = ((unsigned long long)bits << 32) | (unsigned)c;
                    if (key < best) {
                        best = key;
                        best_level = (uint32_t)level;
                    }
                }
            }
            const unsigned long long nearest = wave_min_key(best);
            if (MODE == kTableCodes) {
                if (lane == 0) code[v * M + m] = (uint8_t)nearest;
            } else if (best == nearest && (nearest != ~0ull || lane == 0)) {         // one lane has the nearest pair
                code[(v * M + m) * 2] = nearest == ~0ull ? (uint8_t)0 : (uint8_t)nearest;
                code[(v * M + m) * 2 + 1] = (uint8_t)best_level;
            }
        }
    }
    __syncthreads();
    finish_vectors<kFewRows, WIDE>(g, v0, nv, sel, leaf, code, M * (MODE == kPairCodes ? 2 : 1));
}

template <int MODE>
hipError_t launch_few(const PlaceArgs& a, const FewLds& L, hipStream_t s) {
    const int ds = a.D / a.M;
    const bool wide = reinterpret_cast<uintptr_t>(a.x) % 16 == 0 && ds % 4 == 0;
    const void* fn = wide ? reinterpret_cast<const void*>(place_few_kernel<MODE, true>) : reinterpret_cast<const void*>(place_few_kernel<MODE, false>);
    if (L.total > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)L.total);
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)((a.n + kFewRows - 1) / kFewRows)), block(kFewThreads);
    if (wide) hipLaunchKernelGGL((place_few_kernel<MODE, true>), grid, block, L.total, s, a, L);
    else hipLaunchKernelGGL((place_few_kernel<MODE, false>), grid, block, L.total, s, a, L);
    return hipGetLastError();
}

// Votes with many centroids, whose distances leave room for few wavefronts that have a sub-part each: one workgroup per 64
// vectors and sub-part, its wavefronts share the distances and the pairs.
// pqt_train of 20,000 vectors x 128, 256 centroids, M = 8, five iterations: 19.3 ms; a wavefront per sub-part (two per compute
// unit) 58.1, 44.1 of them for the votes.
template <bool WIDE>
__global__ __launch_bounds__(256) void shared_votes_kernel(PlaceArgs g, int st) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned long long nearest[kPlaceRows];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), waves = blockDim.x / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int m = blockIdx.y;
    const int64_t v0 = (int64_t)blockIdx.x * kPlaceRows;
    const int nv = (int)(g.n - v0 < kPlaceRows ? g.n - v0 : kPlaceRows);
    float* xs = reinterpret_cast<float*>(smem);
    float* at = xs + (size_t)kPlaceRows * st;
    const LinePair* pairs = g.pairs + (size_t)m * g.npairs;
    if (tid < kPlaceRows) nearest[tid] = ~0ull;
    subpart_distances<WIDE, true>(g, v0, nv, m, st, xs, at);
    const int c0 = (int)((int64_t)g.npairs * wave / waves), c1 = (int)((int64_t)g.npairs * (wave + 1) / waves);
    const unsigned long long mine = c0 < c1 ? nearest_line(pairs, c0, c1, at) : ~0ull;
    atomicMin(&nearest[lane], mine);
    __syncthreads();
    if (tid < nv) g.keys[(size_t)m * g.n + v0 + tid] = vote_of(pairs, nearest[tid], m, at);
}

hipError_t launch_shared_votes(const PlaceArgs& a, hipStream_t s) {
    const int ds = a.D / a.M, st = place_layout(ds, a.P, a.k1, 0, 1, true).st;
    const bool wide = reinterpret_cast<uintptr_t>(a.x) % 16 == 0 && ds % 4 == 0;
    const size_t lds = sizeof(float) * ((size_t)kPlaceRows * st + (size_t)a.k1 * kRowStride);
    if (lds > kMaxLds - 1024) return hipErrorInvalidValue;
    const void* fn = wide ? reinterpret_cast<const void*>(shared_votes_kernel<true>) : reinterpret_cast<const void*>(shared_votes_kernel<false>);
    if (lds > 64 * 1024 - 1024) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)((a.n + kPlaceRows - 1) / kPlaceRows), (unsigned)a.M), block(256);
    if (wide) hipLaunchKernelGGL(shared_votes_kernel<true>, grid, block, lds, s, a, st);
    else hipLaunchKernelGGL(shared_votes_kernel<false>, grid, block, lds, s, a, st);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_mode(const PlaceArgs& a, hipStream_t s) {
    const int ds = a.D / a.M, cb = a.M * (MODE == kPairCodes ? 2 : 1);
    const bool wide = reinterpret_cast<uintptr_t>(a.x) % 16 == 0 && ds % 4 == 0;
    if constexpr (MODE != kVotes) {
        const FewLds L = few_layout(ds, a.P, a.k1, a.M, cb);
        if (a.n <= kFewVectors && L.total <= kMaxLds) return launch_few<MODE>(a, L, s);
    }
    // wavefronts per workgroup: those that leave a compute unit the most, none without a sub-part
    int waves = 1;
    size_t most = 0;
    for (int w = 4; w >= 1; w /= 2) {
        const size_t lds = place_layout(ds, a.P, a.k1, cb, w, MODE == kVotes).total;
        if (lds > kMaxLds || (w > a.M && w > 1)) continue;
        const size_t resident = (size_t)w * (kMaxLds / lds);
        if (resident > most) {
            most = resident;
            waves = w;
        }
    }
    const PlaceLds L = place_layout(ds, a.P, a.k1, cb, waves, MODE == kVotes);
    auto launch = [&](auto kernel) {
        if (L.total > 64 * 1024) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)L.total);
            if (e != hipSuccess) return e;
        }
        const dim3 grid((unsigned)((a.n + kPlaceRows - 1) / kPlaceRows)), block((unsigned)waves * kWave);
        hipLaunchKernelGGL(kernel, grid, block, L.total, s, a, L);
        return hipGetLastError();
    };
    // Distances in registers and in LDS, us, 524,288 vectors x 96: k1 = 16 M = 12 527 and 697, M = 24 932 and 1,229; k1 = 32 M = 24 1,591 and
    // 1,861.  Where rows are not read in 16-byte pieces: M = 32 2,237 and 1,926, M = 16 1,600 and 1,413.
    if (!wide) return launch(place_kernel<MODE, false, 0>);
    if (MODE == kTableCodes && a.k1 <= 16) return launch(place_kernel<MODE, true, MODE == kTableCodes ? 16 : 0>);
    if (MODE == kTableCodes && a.k1 <= 32) return launch(place_kernel<MODE, true, MODE == kTableCodes ? 32 : 0>);
    return launch(place_kernel<MODE, true, 0>);
}

// squared norms of the level-1 centroids' sub-parts, added up in double precision as the host does
__global__ void subpart_norms_kernel(const float* C1, int D, int P, int k1, int M, float* c1n) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= M * k1) return;
    const int m = e / k1, i = e - m * k1, dp = D / P, ds = D / M, p = m / (M / P);
    const float* c = C1 + ((size_t)p * k1 + i) * dp + (m * ds - p * dp);
    double s = 0.0;
    for (int d = 0; d < ds; ++d) s = __dadd_rn(s, __dmul_rn((double)c[d], (double)c[d]));
    c1n[e] = (float)s;
}

}  // namespace

hipError_t launch_place(const PlaceArgs& a, bool pair_codes, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    return pair_codes ? launch_mode<kPairCodes>(a, s) : launch_mode<kTableCodes>(a, s);
}

// From more than 32 centroids on (two tiles, whose distances no longer take the staged values' place) the wavefronts share.
hipError_t launch_votes(const PlaceArgs& a, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    return a.k1 > 32 ? launch_shared_votes(a, s) : launch_mode<kVotes>(a, s);
}

hipError_t launch_subpart_norms(const float* C1, int D, int P, int k1, int M, float* c1n, hipStream_t s) {
    hipLaunchKernelGGL(subpart_norms_kernel, dim3((unsigned)((M * k1 + 255) / 256)), dim3(256), 0, s, C1, D, P, k1, M, c1n);
    return hipGetLastError();
}

}  // namespace pqt
