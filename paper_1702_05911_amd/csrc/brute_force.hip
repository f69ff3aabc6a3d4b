// Exact nearest neighbours by brute force (Eq. 1; the paper's "strong baseline" of Table 1): per query the k
// database vectors of smallest squared distance, by (distance, id).  Doubles as the ground truth for recall.
//
// A dense contraction finds the few vectors that can be among the k nearest, and only those get their exact fp32
// distance.  The contraction runs on the bf16 matrix cores, eight times the flops of the fp32 ones: a number is
// cut into bf16 pieces (h = bf16(x), m = bf16(x - h)); byte vectors are one piece exactly.  Byte vectors with queries of bytes
// run on the int8 ones, where everything is exact (filter_as_bytes); the rest of this is about the others.
// With s = ||x||^2 / 2 - q.x (half the squared distance but for the query's own term), the sum of the matrix cores is within
// a ||q|| ||x|| + b ||x||^2 of s: dropped piece products, the rounding of the sums, and the norm (see pqt_host::brute_error).
// 2 ||q|| ||x|| <= ||q||^2 + ||x||^2 parts that, and the filter's value v is the sum less the vector's part (it starts from the
// norm), so that v <= s + a ||q||^2 / 2: the length of one vector widens nothing for the others.  The other way round v is
// at least s less the query's and twice the vector's part, and a vector near the query is at most ||q|| + its
// distance long, so an upper bound of the k-th smallest v gives one of the k-th smallest s, and from that what v may be at
// most for every vector of the true result (keep_up_to).
// Floats often have a common offset, which would count as length: norms and queries are taken relative to a centre c, the
// median of 64 vectors in every dimension.  (q - c).(x - c) differs from (q - c).x by a number that is the same for all
// vectors, so the vectors need not be changed; where the offset is large they are all the same, in registers.  So
//   * the database is walked in chunks, in the order i -> (i * step) mod N with step / N near the golden ratio: every
//     prefix of the order is spread evenly over the database, whatever order the vectors are stored in;
//   * bf_filter_*_kernel contracts a chunk with all queries.  Vectors go from memory through registers, where they are
//     cut, into LDS in the operand layout of v_mfma_f32_32x32x16_bf16 (the queries are laid out once, by
//     pack_queries_kernel): no copy of the database in another format exists.  The first chunk (kDense vectors) is written
//     out; from then on only pairs whose value may matter are kept: the accumulators start from the norm, a maximum of 16
//     values and one comparison decide for 16 pairs, and a lane appends what passes to a list of its own, so that no
//     counter is shared (a query belongs to one column of one wavefront);
//   * bf_select_kernel, one workgroup per query, bounds the k-th smallest value by a 1024-bin histogram and keeps what
//     can still matter; after the last chunk it computes the exact distances sum (y - x)^2 of that list
//     (k and a few more) in fp32 and sorts them.
// What a vector's value may be at most is a guess between chunks: of the k nearest, about k p are among the first p N vectors, and
// hardly ever more than rank_at() says, six deviations more; the bound is that of the rank-th smallest value so far, not of
// the k-th.  It never grows, so the list always holds everything up to it, and if in the end k values are
// up to it, those nearest were all kept; if not, the query is searched as one whose lists overflow.  A third of the pairs pass
// that the k-th smallest value lets through (10,000 queries x 1M x 128 bytes, k = 100: 2.35 -> 1.8 ms).
// A query whose lists
// overflow (more than about two thousand vectors tied with the k-th, or non-finite data) is searched by bf_scan_kernel, exact
// distances to all vectors.
//
// Measured, 10,000 queries x 1M x 128 bytes, k = 100: 1.8 ms (the contraction 1.45, selection
// 0.35); as one bf16 piece, all up to the k-th smallest so far kept, 3.5 ms (contraction 3.0), with
// the fp32 matrix cores and all distances written and read back 40.0 ms.  777 x 150,001 x 960 floats, k = 10:
// 0.52 ms (contraction 0.47; by bf16 pieces 0.80 and 0.73) against 2.58; 3 x 901,800 x 128 bytes: 0.15 against 0.71.
// Data on which a bound by the largest norm of all, a list of 2 k + 256 and a scan by one workgroup per query took 78 ms
// (the same floats, 777 queries; fp32 matrix cores 2.7): one vector of norm 300 among unit vectors 1.0 ms, an offset of 10 1.0,
// 1,000 copies of one vector 1.2.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "pqt_device.hpp"
#include "pqt_host.hpp"
#include "pqt_kernels.hpp"
#include "row_distance.hpp"

namespace pqt {
namespace {

typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16v8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfv8 __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));    // (arrays of HIP's uint4 end up in scratch memory)

constexpr int kBfThreads = 256;
constexpr int kDense = 4096;           // vectors of the first chunk; also the entries a select workgroup holds in LDS
constexpr int kFrag = 512;             // bf16 values of one fragment: 32 rows x 16 dimensions
constexpr int kStatRows = 64;          // database vectors per LDS tile of the stationary kernel, as bf16 ...
constexpr int kByteRows = 128;         // ... and as bytes
constexpr int kStatQueries = 512;      // queries of one of its workgroups
// a query tile's state: second bf16 pieces; values that are not 0 .. 255; a norm out of the halves' range
constexpr uint32_t kSecondPiece = 1u, kNotBytes = 2u, kNoHalves = 4u;
constexpr uint32_t kHalvesOff = 1u << 31;        // control[kBfCrowded]: no halves for this call, however many queries are crowded
constexpr float kHalfNorms = 0x1p40f;  // norms within this and its reciprocal are scaled to 2^14 .. 2^15 for the halves
constexpr int kGenRows = 256, kGenQueries = 128;   // workgroup tile of the general kernel ...
constexpr int kHalfQueries = 256;      // ... and the queries of one of the kernel for halves

__device__ __forceinline__ v16f mfma(bf16x8 a, bf16x8 b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16v8, a), __builtin_bit_cast(bf16v8, b), c, 0, 0, 0);
}

__global__ void clear_words_kernel(uint32_t* out) { out[threadIdx.x] = 0u; }

__device__ __forceinline__ uint32_t pack2(float a, float b) {      // two floats to bf16, nearest even
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ v16f mfma_half(bf16x8 a, bf16x8 b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfv8, a), __builtin_bit_cast(halfv8, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t pack2_half(float a, float b) {         // two floats to half precision, nearest even
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, f16x2));
}
// the power of two that takes a norm to 2^14 .. 2^15 (1 for zero)
__device__ __forceinline__ float half_scale(float norm) {
    return norm > 0.0f ? __uint_as_float((uint32_t)(127 + 14 + 127 - (int)(__float_as_uint(norm) >> 23)) << 23) : 1.0f;
}
__device__ __forceinline__ bool half_norm_ok(float norm) { return norm == 0.0f || (norm >= 1.0f / kHalfNorms && norm <= kHalfNorms); }
__device__ __forceinline__ float low_value(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float high_value(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }

// Queries -> fragments of two pieces (h, then m): one workgroup per tile of 32 queries, its wavefronts share the steps of
// 16 dimensions (16 of them where there are many steps); lane l holds query l % 32, dimensions 8 * (l / 32) .. + 8 of a step.
// Also ||q||, whether a query of the tile has a second piece that is not zero or is not all bytes, and the state of the call: no
// query is left to the exact scan.  qbytes (stationary kernel): the values less 128 as they are if they are bytes, in the operand
// layout of v_mfma_i32_32x32x32_i8, lane l with query l % 32, dimensions 16 * (l / 32) .. + 16 of a step of 32.
__global__ __launch_bounds__(1024) void pack_queries_kernel(BruteArgs g) {
    __shared__ float red[2][1024 / kWave][32];
    __shared__ uint32_t state;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, nwaves = (int)blockDim.x / kWave, D = g.D, KS = g.KS;
    if (tid == 0) {
        state = 0u;
        if (blockIdx.x == 0) g.control[kBfTodo] = g.control[kBfCrowded] = 0u;
    }
    __syncthreads();
    const int64_t tile = blockIdx.x, q = tile * 32 + (lane & 31);
    const bool have = q < g.nq;
    const float* row = g.queries + (have ? (size_t)q * D : 0);
    float norm = 0.0f, shift = 0.0f;
    uint32_t second = 0;
    bool bytes = true;
#pragma unroll 4
    for (int ks = wave; ks < KS; ks += nwaves) {
        const int d = have ? ks * 16 + 8 * (lane >> 5) : D;               // D is a multiple of four
        const float4 z = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        const float4 v0 = d < D ? *reinterpret_cast<const float4*>(row + d) : z;
        const float4 v1 = d + 4 < D ? *reinterpret_cast<const float4*>(row + d + 4) : z;
        float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        if (g.centre) {                                      // (zeros where it is not used)
            const float4 c0 = d < D ? *reinterpret_cast<const float4*>(g.centre + d) : z;
            const float4 c1 = d + 4 < D ? *reinterpret_cast<const float4*>(g.centre + d + 4) : z;
            v[0] -= c0.x; v[1] -= c0.y; v[2] -= c0.z; v[3] -= c0.w;
            v[4] -= c1.x; v[5] -= c1.y; v[6] -= c1.z; v[7] -= c1.w;
            shift = fmaf(v[0], c0.x, fmaf(v[1], c0.y, fmaf(v[2], c0.z, fmaf(v[3], c0.w, shift))));
            shift = fmaf(v[4], c1.x, fmaf(v[5], c1.y, fmaf(v[6], c1.z, fmaf(v[7], c1.w, shift))));
        }
        u32x4 h, m;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            norm = fmaf(v[2 * c + 1], v[2 * c + 1], fmaf(v[2 * c], v[2 * c], norm));
            h[c] = pack2(v[2 * c], v[2 * c + 1]);
            m[c] = pack2(v[2 * c] - low_value(h[c]), v[2 * c + 1] - high_value(h[c]));
            second |= m[c] & 0x7fff7fffu;
        }
        u32x4* out = reinterpret_cast<u32x4*>(g.qfrag) + (tile * KS + ks) * (2 * kFrag / 8) + lane;
        out[0] = h;
        out[kFrag / 8] = m;
        if (g.qbytes) {
            uint32_t packed[2] = {0u, 0u};
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const bool is_byte = v[c] >= 0.0f && v[c] <= 255.0f && v[c] == truncf(v[c]);
                bytes = bytes && is_byte;
                const uint32_t b = is_byte && d + c < D ? ((uint32_t)v[c] & 0xffu) ^ 0x80u : 0u;       // (nothing past the last dimension)
                packed[c / 4] |= b << (8 * (c % 4));
            }
            reinterpret_cast<uint2*>(g.qbytes)[((tile * (KS / 2) + ks / 2) * kWave + (ks & 1) * 32 + (lane & 31)) * 2 + (lane >> 5)] =
                make_uint2(packed[0], packed[1]);
        }
    }
    norm += __shfl_xor(norm, 32, kWave);
    shift += __shfl_xor(shift, 32, kWave);
    if (lane < 32) {
        red[0][wave][lane] = norm;
        red[1][wave][lane] = shift;
    }
    const uint32_t found = (__any(second != 0) ? kSecondPiece : 0u) | (__any(!bytes) ? kNotBytes : 0u);
    if (lane == 0 && found) atomicOr(&state, found);
    __syncthreads();
    if (tid < 32) {
        float n2 = 0.0f, c = 0.0f;
        for (int w = 0; w < nwaves; ++w) {
            n2 += red[0][w][tid];
            c += red[1][w][tid];
        }
        g.qnorm[q] = sqrtf(n2);
        g.qshift[q] = g.use_centre[0] ? 0.0f : c;
        g.flagged[q] = 0u;
        g.scan_done[q] = 0u;
        if (g.qhalf && (!half_norm_ok(sqrtf(n2)) || !half_norm_ok(g.xhalf[g.N] + g.xhalf[g.N + 2]))) atomicOr(&state, kNoHalves);
    }
    if (g.qhalf) __syncthreads();
    if (tid == 0) g.second[tile] = state;
}

// Queries relative to the centre -> fragments of one piece of half precision, scaled.  A thread per eight dimensions.
__global__ __launch_bounds__(kBfThreads) void pack_halves_kernel(BruteArgs g, int64_t count) {
    const int64_t e = (int64_t)blockIdx.x * kBfThreads + threadIdx.x;
    if (e >= count) return;
    const int lane = (int)(e % kWave), ks = (int)(e / kWave % g.KS), D = g.D, d = ks * 16 + 8 * (lane >> 5);
    const int64_t q = e / kWave / g.KS * 32 + (lane & 31);
    const float* row = g.queries + (q < g.nq ? (size_t)q * D : 0);
    const float scale = half_scale(g.qnorm[q]);
    u32x4 h = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int c = 0; c < 2; ++c)
        if (q < g.nq && d + 4 * c < D) {                     // D is a multiple of four
            const float4 v = *reinterpret_cast<const float4*>(row + d + 4 * c), m = *reinterpret_cast<const float4*>(g.centre + d + 4 * c);
            h[2 * c] = pack2_half((v.x - m.x) * scale, (v.y - m.y) * scale);
            h[2 * c + 1] = pack2_half((v.z - m.z) * scale, (v.w - m.w) * scale);
        }
    reinterpret_cast<u32x4*>(g.qhalf)[e] = h;
}

// The centre of float vectors: in every dimension the median of 64 vectors spread over the database (places 0 .. 63 of the
// database order), which a few long ones do not move.  64 dimensions per workgroup.
constexpr int kCentreRows = 64;
__global__ __launch_bounds__(kBfThreads) void centre_kernel(const float* x, uint64_t N, uint64_t step, int D, float* centre) {
    constexpr int kWaves = kBfThreads / kWave, kPer = kCentreRows / kWaves;
    __shared__ uint32_t key[kCentreRows][kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, d = blockIdx.x * kWave + lane;
    float mine[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        mine[u] = x[((uint64_t)(wave + u * kWaves) * step % N) * (uint64_t)D + (d < D ? d : 0)];
#pragma unroll
    for (int u = 0; u < kPer; ++u) key[wave + u * kWaves][lane] = mono_key(mine[u]);
    __syncthreads();
    int below[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) below[u] = 0;
    for (int o = 0; o < kCentreRows; ++o) {
        const uint32_t other = key[o][lane];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const uint32_t own = mono_key(mine[u]);
            below[u] += other < own || (other == own && o < wave + u * kWaves) ? 1 : 0;
        }
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (below[u] == kCentreRows / 2 && d < D) centre[d] = fabsf(mine[u]) < 1e18f ? mine[u] : 0.0f;
}

// How the centre is used, from the norms of the same vectors with and without it: not at all (it becomes zero) unless it takes
// two thirds off the squared norms of most of them, 48 of the 64; subtracted from the vectors too (*use = 1) where
// it takes 24 of 25 parts off, which costs the contraction 10 to 15 % (in small batches more), and otherwise the values'
// window grows with the centre's norm (*mu).  One workgroup.
__global__ __launch_bounds__(1024) void use_centre_kernel(const float* x, uint64_t N, uint64_t step, int D, float* centre, uint32_t* use, float* mu) {
    __shared__ uint32_t shorter[2];
    __shared__ float square[1024 / kWave];
    constexpr int kWaves = 1024 / kWave, kPer = kCentreRows / kWaves;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (threadIdx.x < 2) shorter[threadIdx.x] = 0u;
    __syncthreads();
    const float* row[kPer];
    float with[kPer], without[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        row[u] = x + ((uint64_t)(wave + u * kWaves) * step % N) * (uint64_t)D;
        with[u] = without[u] = 0.0f;
    }
#pragma unroll 4
    for (int d = lane; d < D; d += kWave) {
        const float at = centre[d];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const float v = row[u][d];
            with[u] = fmaf(v - at, v - at, with[u]);
            without[u] = fmaf(v, v, without[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        for (int off = 1; off < kWave; off <<= 1) {
            with[u] += __shfl_xor(with[u], off, kWave);
            without[u] += __shfl_xor(without[u], off, kWave);
        }
        if (lane == 0 && 3.0f * with[u] < without[u]) atomicAdd(&shorter[0], 1u);
        if (lane == 0 && 25.0f * with[u] < without[u]) atomicAdd(&shorter[1], 1u);
    }
    float own = 0.0f;
    for (int d = threadIdx.x; d < D; d += 1024) own = fmaf(centre[d], centre[d], own);
    for (int off = 1; off < kWave; off <<= 1) own += __shfl_xor(own, off, kWave);
    if (lane == 0) square[wave] = own;
    __syncthreads();
    const bool any = shorter[0] >= kCentreRows * 3 / 4, all = shorter[1] >= kCentreRows * 3 / 4;
    if (!any)
        for (int d = threadIdx.x; d < D; d += 1024) centre[d] = 0.0f;
    if (threadIdx.x == 0) {
        float sum = 0.0f;
        for (int w = 0; w < kWaves; ++w) sum += square[w];
        *use = any && all ? 1u : 0u;
        *mu = any && !all ? 1.001f * sqrtf(sum) : 0.0f;
    }
}

// What the accumulators start from, the half squared norms of the database vectors less their part of the error bound, and, in the
// word behind them, the bits of the largest norm (a little enlarged; never negative, so bits order as values).  A group of
// lanes per row, 16 bytes per lane and step.
// Bytes: in `whole` the same of the vectors less 128, rounded down to a whole number.  Floats: in `out_half` the same for the products
// of halves.
template <typename Elem>
__global__ __launch_bounds__(kBfThreads) void half_norms_kernel(const Elem* x, int64_t n, int D, const float* centre, pqt_host::BruteError err, pqt_host::BruteError half, float* out, int* whole, float* out_half) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    constexpr int pe = 16 / (int)sizeof(Elem);
    const int npieces = D / pe, lpr = lanes_per_row(npieces), per_wave = kWave / lpr, sub = lane / lpr, l = lane & (lpr - 1);
    const int64_t nwaves = (int64_t)gridDim.x * (kBfThreads / kWave);
    float top = 0.0f;
    bool as_they_are = false;                  // the filter's products are with vectors that are not centred
    if constexpr (sizeof(Elem) == 4) as_they_are = out[n + 2] != 0.0f;
    for (int64_t r0 = ((int64_t)blockIdx.x * (kBfThreads / kWave) + wave) * per_wave; r0 < n; r0 += nwaves * per_wave) {
        const int64_t r = r0 + sub;
        float s = 0.0f, raw = 0.0f;
        int signed_norm = 0;
        if (r < n) {
#pragma unroll 4
            for (int piece = l; piece < npieces; piece += lpr) {
                const u32x4 w = reinterpret_cast<const u32x4*>(x + (size_t)r * D)[piece];
                u32x4 c = {0u, 0u, 0u, 0u};
                if constexpr (sizeof(Elem) == 4) c = reinterpret_cast<const u32x4*>(centre)[piece];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if constexpr (sizeof(Elem) == 4) {
                        const float v = __uint_as_float(w[j]) - __uint_as_float(c[j]);
                        s = fmaf(v, v, s);
                        raw = fmaf(__uint_as_float(w[j]), __uint_as_float(w[j]), raw);
                    } else {
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const float v = (float)((w[j] >> (8 * b)) & 0xffu);
                            s = fmaf(v, v, s);
                        }
                        const int less = (int)(w[j] ^ 0x80808080u);
                        signed_norm = __builtin_amdgcn_sdot4(less, less, signed_norm, false);
                    }
                }
            }
        }
        for (int off = 1; off < lpr; off <<= 1) {
            s += __shfl_xor(s, off, kWave);
            if constexpr (sizeof(Elem) == 4) raw += __shfl_xor(raw, off, kWave);
            else signed_norm += __shfl_xor(signed_norm, off, kWave);
        }
        if (sizeof(Elem) == 1 && r < n && l == 0) whole[r] = signed_norm >> 1;
        if (r < n && l == 0) out[r] = (0.5f - err.norm) * s - 0.5f * err.dot * (as_they_are ? raw : s);
        if (sizeof(Elem) == 4 && r < n && l == 0) out_half[r] = (0.5f - half.norm) * s - 0.5f * half.dot * (as_they_are ? raw : s);
        top = fmaxf(top, r < n ? s : 0.0f);
        if (r < n && s != s) top = __builtin_inff();
    }
    // (one atomic per workgroup: one per wavefront took longer than the rest)
    __shared__ uint32_t wave_top[kBfThreads / kWave];
    const uint32_t bits = wave_max_u32(__float_as_uint(1.001f * sqrtf(top)));
    if (lane == 0) wave_top[wave] = bits;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t most = bits;
        for (int w = 1; w < kBfThreads / kWave; ++w) most = max(most, wave_top[w]);
        atomicMax(reinterpret_cast<uint32_t*>(out) + n, most);
    }
}

// What the value of a vector of the true result may be at most, when k vectors seen have values of at most v.
// Norms are relative to the centre; mu, the norm of the centre, joins them where products are with vectors as they are, and
// `shift` = (q - c).c turns a value into one of centred vectors.  The k-th smallest s is at most v + own + e(r), `own` the query's
// part, e(r) twice the part of a vector of norm r, r the largest norm that a vector with value v can have: s >= r^2 / 2 - qn r
// gives r <= qn + sqrt(qn^2 + 2 (v + shift + own + e(r))), which is applied again and again from the largest norm of all.
// A query longer than all vectors has the tighter a ||q|| X for its part, X the largest norm.  0.1 % on r and 3 % on the sum for
// the rounding here.
__device__ __forceinline__ float keep_up_to(const BruteArgs& g, const pqt_host::BruteError& err, float qn, float shift, float v) {
    const float top = g.xhalf[g.N], mu = g.xhalf[g.N + 2];
    const float own = 0.5f * err.dot * qn * fminf(qn, 2.0f * (top + mu)) + err.flush * qn * (top + mu) + pqt_host::kBruteUnderflow;
    float r = top, e = 0.0f;
    for (int i = 0; i < 6; ++i) {
        e = err.dot * (r + mu) * (r + mu) + 2.0f * err.norm * r * r;
        const float t = qn * qn + 2.0f * (v + shift + own + e + err.dot * qn * mu);
        r = fminf(r, 1.001f * (qn + sqrtf(fmaxf(t, 0.0f))));
    }
    return v + 1.03f * (2.0f * own + e);
}

// What an accumulator has to reach to be kept, from what bf_select_kernel left of a query
__device__ __forceinline__ float keep_from(const BruteArgs& g, const float* keep, int64_t q) {
    return q >= g.nq || g.flagged[q] ? __builtin_inff() : -keep[q];
}

// Floats, after the first chunk: are the values of these queries those of products of halves?
__device__ __forceinline__ bool call_is_halves(const BruteArgs& g) { return g.qhalf && g.control[kBfCrowded] <= g.crowded_most; }

// What the queries of this group of the stationary kernel are, and whether they are all whole numbers 0 .. 255.
__device__ __forceinline__ uint32_t query_state(const BruteArgs& g, int group) {
    uint32_t state = 0;
#pragma unroll
    for (int tile = 0; tile < kStatQueries / 32; ++tile) state |= g.second[group * (kStatQueries / 32) + tile];
    return state;
}
__device__ __forceinline__ bool group_is_bytes(const BruteArgs& g, int group) { return !(query_state(g, group) & kNotBytes); }

// One 32 x 32 tile of accumulators: lane l holds query column l % 32 and database rows 8 * (r / 4) + 4 * (l / 32) + r % 4.
// DENSE: all values go to out (s~ of the query's row of kDense values).  Else those that reach `from` are appended to the
// lane's list (row of the chunk, s~); a maximum of four rows says whether to look at each.
template <typename Value>
__device__ __forceinline__ Value larger(Value a, Value b) {
    if constexpr (std::is_same<Value, float>::value) return fmaxf(a, b);
    else return a > b ? a : b;
}
// unscale: what takes a sum to a value.
template <bool DENSE, typename Acc, typename Value>
__device__ __forceinline__ void take_tile(const Acc& acc, Value from, uint32_t row0, float* dense, uint2* list, int cap, uint32_t& count,
                                          float unscale = 1.0f) {
    if (DENSE) {
        if (!dense) return;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<float4*>(dense + row0 + 8 * i) = make_float4((float)-acc[4 * i], (float)-acc[4 * i + 1], (float)-acc[4 * i + 2], (float)-acc[4 * i + 3]);
        return;
    }
    Value four[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) four[i] = larger(larger(acc[4 * i], acc[4 * i + 1]), larger(acc[4 * i + 2], acc[4 * i + 3]));
    if (larger(larger(four[0], four[1]), larger(four[2], four[3])) >= from) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (four[i] >= from) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (acc[4 * i + c] >= from) {
                        list[count < (uint32_t)cap ? count : cap - 1] = make_uint2(row0 + 8 * i + c, __float_as_uint((float)-acc[4 * i + c] * unscale));
                        ++count;
                    }
            }
    }
}

// Workgroups go to the eight chiplets in turn; the query groups that read the same database tiles are put on one chiplet,
// one after the other, so that its L2 holds a tile for all of them (splits a multiple of eight; else in plain order).
__device__ __forceinline__ void place_of_workgroup(int b, int splits, int groups, int& split, int& group) {
    if (splits % 8) {
        split = b % splits;
        group = b / splits;
    } else {
        const int l = b / 8;
        group = l % groups;
        split = l / groups * 8 + b % 8;
    }
}

// The rows of the database tiles a workgroup of the kernels below brings into LDS: tiles of up to ROWS vectors, every splits-th
// of the chunk, as 16-byte pieces (KS of them, 16 dimensions each) that a thread has the same places of in every tile.
template <int KS, int ROWS>
struct TileRows {
    static constexpr int kPieces = (ROWS * KS + kBfThreads - 1) / kBfThreads;           // pieces per thread
    int row[kPieces], step[kPieces];           // piece i is step[i] of row[i]
    bool mine[kPieces];
    u32x4 piece[kPieces];
    uint64_t at[kPieces], hid, move;           // where in the database those pieces are; the vector of row tid
    int D16;
    __device__ __forceinline__ void start(const BruteArgs& g, int split, int tile_rows) {
        const int tid = threadIdx.x;
        D16 = g.D / 16;
        move = ((uint64_t)g.splits * tile_rows) % g.N * g.step % g.N;
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int e = i * kBfThreads + tid;
            // rows four apart within a wavefront's instruction, so that row ^ step takes all sixteen bank groups
            const int r = e / KS;
            step[i] = e - r * KS;
            row[i] = KS == 8 ? (r & ~31) | (r & 7) << 2 | (r >> 3 & 3) : r & (ROWS - 1);
            mine[i] = e < ROWS * KS && row[i] < tile_rows;
            at[i] = ((g.chunk_pos + (uint64_t)split * tile_rows + row[i]) % g.N) * g.step % g.N * (uint64_t)g.D + (step[i] < D16 ? step[i] * 16 : 0);
        }
        hid = ((g.chunk_pos + (uint64_t)split * tile_rows + (tid & (ROWS - 1))) % g.N) * g.step % g.N;
    }
    // the next tile's pieces, then the ids move on; past the last tile: some vectors, unused (always loading keeps the pieces in
    // registers).  Returns the vector of row tid.
    __device__ __forceinline__ uint64_t fetch(const BruteArgs& g) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const u32x4 zero = {0u, 0u, 0u, 0u};
            const u32x4 v = *reinterpret_cast<const u32x4*>(static_cast<const uint8_t*>(g.vectors) + at[i]);
            piece[i] = step[i] < D16 ? v : zero;
            at[i] += move * (uint64_t)g.D;
            at[i] -= at[i] >= g.N * (uint64_t)g.D ? g.N * (uint64_t)g.D : 0;       // (a piece lies less than D behind its vector's start)
        }
        const uint64_t h = hid;
        hid += move;
        hid -= hid >= g.N ? g.N : 0;
        return h;
    }
};

// Byte vectors of at most 128 dimensions, queries that are not all bytes: a wavefront keeps 64 queries (KS steps,
// two pieces, or one where the group has no more than 256 queries), or 128 of one piece, in registers for the whole launch, and the
// workgroup's 256 or 512 share the database tiles that stream through LDS, two in turn.  (67 queries of one piece, 1M x 128, k = 10: 145 us
// with 128 a wavefront, one of four at work, 118 with 64.)
// LDS: 16 bytes of (row, step, half) lie in slot row ^ step of the fragment's half: eight lanes bring a row's eight steps
// and would all hit the same banks.
template <int KS, int QP, int NC, bool DENSE>
__device__ __forceinline__ void filter_as_bf16(const BruteArgs& g, unsigned char* smem, int split, int64_t first_query) {
    constexpr int kTileBytes = kStatRows / 32 * KS * kFrag * 2;                // NC: tiles of 32 queries a wavefront has
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, splits = g.splits;
    const int64_t q0 = first_query + wave * (NC * 32);
    const bool active = q0 < g.nq;             // (else the wavefront only brings vectors)
    bf16x8 bq[QP][NC][KS];
    float from[NC];
    uint32_t count[NC];
#pragma unroll
    for (int ct = 0; ct < NC; ++ct) {
        count[ct] = 0;
#pragma unroll
        for (int p = 0; p < QP; ++p)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                bq[p][ct][ks] = reinterpret_cast<const bf16x8*>(g.qfrag)[((q0 / 32 + ct) * KS + ks) * (2 * kFrag / 8) + p * (kFrag / 8) + lane];
        from[ct] = DENSE ? 0.0f : keep_from(g, g.keep, q0 + ct * 32 + (lane & 31));
    }
    const int ntile = (int)((g.chunk_rows + kStatRows - 1) / kStatRows);
    TileRows<KS, kStatRows> rows;
    rows.start(g, split, kStatRows);
    float hx = 0.0f;
    auto fetch = [&](int t) {
        const uint64_t h = rows.fetch(g);
        hx = (int64_t)t * kStatRows + (tid & (kStatRows - 1)) < g.chunk_rows ? g.xhalf[h] : __builtin_inff();   // such rows enter no list
    };
    fetch(split);
    int buf = 0;
    for (int t = split; t < ntile; t += splits, buf ^= 1) {
        u32x4* xs = reinterpret_cast<u32x4*>(smem + buf * kTileBytes);
        float* hs = reinterpret_cast<float*>(smem + 2 * kTileBytes) + buf * kStatRows;
#pragma unroll
        for (int i = 0; i < TileRows<KS, kStatRows>::kPieces; ++i) {
            u32x4 w0, w1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t b = rows.piece[i][j];
                const uint32_t p0 = pack2((float)(b & 0xffu), (float)((b >> 8) & 0xffu)), p1 = pack2((float)((b >> 16) & 0xffu), (float)(b >> 24));
                if (j < 2) { w0[2 * j] = p0; w0[2 * j + 1] = p1; }
                else { w1[2 * j - 4] = p0; w1[2 * j - 3] = p1; }
            }
            const uint32_t r = (uint32_t)rows.row[i], ks = (uint32_t)rows.step[i];
            const uint32_t slot = ((r >> 5) * KS + ks) * 64u + ((r & 31u) ^ ks);
            if (rows.mine[i]) {
                xs[slot] = w0;
                xs[slot + 32] = w1;
            }
        }
        if (tid < kStatRows) hs[tid] = -hx;
        __syncthreads();                       // the tile before the last is read by nobody any more: one barrier per tile
        fetch(t + splits);
        if (!active) continue;
#pragma unroll 1
        for (int rt = 0; rt < kStatRows / 32; ++rt) {
            const uint32_t row0 = (uint32_t)t * kStatRows + rt * 32 + 4 * (lane >> 5);
#pragma unroll
            for (int c2 = 0; c2 < NC; c2 += 2) {
                if (c2 && q0 + c2 * 32 >= g.nq) break;
                asm volatile("" ::: "memory");               // (read from LDS again: both halves' operands do not fit the registers)
                v16f c;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 h = *reinterpret_cast<const float4*>(&hs[rt * 32 + 8 * i + 4 * (lane >> 5)]);
                    c[4 * i] = h.x; c[4 * i + 1] = h.y; c[4 * i + 2] = h.z; c[4 * i + 3] = h.w;
                }
                v16f acc[2] = {c, c};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const bf16x8 a = reinterpret_cast<const bf16x8*>(xs)[(rt * KS + ks) * (kFrag / 8) + (lane ^ ks)];
#pragma unroll
                    for (int p = 0; p < QP; ++p) {
                        acc[0] = mfma(a, bq[p][c2][ks], acc[0]);
                        acc[1] = mfma(a, bq[p][c2 + 1][ks], acc[1]);
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int64_t q = q0 + (c2 + u) * 32 + (lane & 31);
                    take_tile<DENSE>(acc[u], from[c2 + u], row0, DENSE && q < g.nq ? g.dense + (size_t)q * kDense : nullptr,
                                     g.lists + ((size_t)q * g.segs + split * 2 + (lane >> 5)) * g.seg_cap, g.seg_cap, count[c2 + u]);
                }
            }
        }
    }
    if (DENSE || !active) return;
#pragma unroll
    for (int ct = 0; ct < NC; ++ct)
        g.seg_count[(size_t)(q0 + ct * 32 + (lane & 31)) * g.segs + split * 2 + (lane >> 5)] = count[ct];
}

// Byte vectors of at most 128 dimensions and queries of bytes: both less 128, which changes no distance, on the int8 matrix cores at
// twice the bf16 rate, exactly.  A wavefront keeps 128 queries in registers, the workgroup's 512 share the database
// tiles that stream through LDS as they are in memory but for the sign bit, two in turn.
// Per 32 vectors a wavefront reads 4 KB of fragments and 4 of what the sums start from for 16 matrix instructions of 32 cycles:
// half the LDS rate.  The sums of 64 queries are looked at (eight maxima per 16) while the next 64 queries' are formed, three vector
// instructions behind each matrix instruction.  488,000 vectors x 10,000 queries that pass nothing: 493 us, 2.5 P operations a
// second (maxima behind the matrix instructions: 525; without the loads 450, the matrix cores busy 62 % at the 2.0 GHz the
// card then runs at).
template <int KS, bool DENSE>
__device__ __forceinline__ void filter_as_bytes(const BruteArgs& g, unsigned char* smem, int split, int64_t first_query) {
    constexpr int KB = KS / 2, NC = 4, kTileBytes = kByteRows * KS * 16;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, splits = g.splits;
    const int64_t q0 = first_query + wave * (NC * 32);
    const bool active = q0 < g.nq;             // (else the wavefront only brings vectors)
    i32x4 bq[NC][KB];
    int from[NC];
    uint32_t count[NC];
#pragma unroll
    for (int ct = 0; ct < NC; ++ct) {
        count[ct] = 0;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) bq[ct][kb] = reinterpret_cast<const i32x4*>(g.qbytes)[((q0 / 32 + ct) * KB + kb) * kWave + lane];
        const float f = DENSE ? 0.0f : keep_from(g, g.keep, q0 + ct * 32 + (lane & 31));
        from[ct] = f < 1e9f ? (int)ceilf(f) : 0x7fffffff;                     // (values are whole)
    }
    auto take = [&](const v16i& acc, auto ct, uint32_t row0) {
        const int64_t q = q0 + ct * 32 + (lane & 31);
        take_tile<DENSE>(acc, from[ct], row0, DENSE && q < g.nq ? g.dense + (size_t)q * kDense : nullptr,
                         g.lists + ((size_t)q * g.segs + split * 2 + (lane >> 5)) * g.seg_cap, g.seg_cap, count[ct]);
    };
    auto largest = [](const v16i& acc) {
        int top = larger(acc[0], acc[1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) top = larger(larger(acc[r], acc[r + 1]), top);
        return top;
    };
    constexpr std::integral_constant<int, 0> c0;
    constexpr std::integral_constant<int, 2> c2;
    constexpr std::integral_constant<int, 3> c3;
    const int tile_rows = g.tile_rows, ntile = (int)((g.chunk_rows + tile_rows - 1) / tile_rows);
    TileRows<KS, kByteRows> rows;
    rows.start(g, split, tile_rows);
    int hx = 0;
    auto fetch = [&](int t) {
        const uint64_t h = rows.fetch(g);
        hx = (int64_t)t * tile_rows + (tid & (kByteRows - 1)) < g.chunk_rows ? g.ihalf[h] : 0x40000000;   // such rows enter no list
    };
    fetch(split);
    v16i acc[NC];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[2][r] = acc[3][r] = -0x7fffffff;         // (nothing to look at yet)
    uint32_t row0 = 0;                                                       // of acc[2] and acc[3]
    bool none = true;
    int buf = 0;
    for (int t = split; t < ntile; t += splits, buf ^= 1) {
        u32x4* xs = reinterpret_cast<u32x4*>(smem + buf * kTileBytes);
        int* hs = reinterpret_cast<int*>(smem + 2 * kTileBytes) + buf * kByteRows;
#pragma unroll
        for (int i = 0; i < TileRows<KS, kByteRows>::kPieces; ++i) {
            const uint32_t r = (uint32_t)rows.row[i], ks = (uint32_t)rows.step[i];
            if (rows.mine[i]) xs[((r >> 5) * KS + ks) * 32u + ((r & 31u) ^ ks)] = rows.piece[i] ^ 0x80808080u;
        }
        if (tid < kByteRows) hs[tid] = -hx;
        __syncthreads();                       // the tile before the last is read by nobody any more: one barrier per tile
        fetch(t + splits);
        if (!active) continue;
#pragma unroll 1
        for (int rt = 0; rt < tile_rows / 32; ++rt) {
            i32x4 a[KB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)    // half h of step kb is piece 2 kb + h of its row
                a[kb] = reinterpret_cast<const i32x4*>(xs)[(rt * KB + kb) * kWave + (lane ^ (2 * kb + (lane >> 5)))];
            v16i c;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const i32x4 h = *reinterpret_cast<const i32x4*>(&hs[rt * 32 + 8 * i + 4 * (lane >> 5)]);
                c[4 * i] = h[0]; c[4 * i + 1] = h[1]; c[4 * i + 2] = h[2]; c[4 * i + 3] = h[3];
            }
            // sums of tiles ct and ct + 1; meanwhile the largest of tiles was and was + 1
            auto form = [&](auto ct, auto was, uint32_t was_row0, bool look) {
                acc[ct] = c;
                acc[ct + 1] = c;
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    acc[ct] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[kb], bq[ct][kb], acc[ct], 0, 0, 0);
                    acc[ct + 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[kb], bq[ct + 1][kb], acc[ct + 1], 0, 0, 0);
                }
                const int x = largest(acc[was]), y = largest(acc[was + 1]);
                const bool found = DENSE ? look : (x >= from[was]) | (y >= from[was + 1]);
#pragma unroll
                for (int i = 0; i < 2 * KB; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
                }
                if (found) {
                    take(acc[was], was, was_row0);
                    take(acc[was + 1], std::integral_constant<int, was + 1>{}, was_row0);
                }
            };
            form(c0, c2, row0, !none);
            none = false;
            row0 = (uint32_t)t * tile_rows + rt * 32 + 4 * (lane >> 5);
            form(c2, c0, row0, true);
        }
    }
    if (!active) return;
    if (!none) {
        take(acc[2], c2, row0);
        take(acc[3], c3, row0);
    }
    if (!DENSE) {
#pragma unroll
        for (int ct = 0; ct < NC; ++ct)
            g.seg_count[(size_t)(q0 + ct * 32 + (lane & 31)) * g.segs + split * 2 + (lane >> 5)] = count[ct];
    }
}

template <int KS, bool DENSE>
__global__ __launch_bounds__(kBfThreads, 2) void bf_filter_stationary_kernel(BruteArgs g) {
    constexpr int kTileBytes = kStatRows * KS * 32 > kByteRows * KS * 16 ? kStatRows * KS * 32 : kByteRows * KS * 16;
    constexpr int kNorms = kStatRows > kByteRows ? kStatRows : kByteRows;
    __shared__ __align__(16) unsigned char smem[2 * kTileBytes + 2 * kNorms * sizeof(float)];
    int split, group;
    place_of_workgroup(blockIdx.x, g.splits, (int)gridDim.x / g.splits, split, group);
    const int64_t first_query = (int64_t)group * kStatQueries;
    if (group_is_bytes(g, group)) {
        filter_as_bytes<KS, DENSE>(g, smem, split, first_query);
        return;
    }
    if (!(query_state(g, group) & kSecondPiece)) {
        if (g.nq - first_query > kStatQueries / 2) filter_as_bf16<KS, 1, 4, DENSE>(g, smem, split, first_query);
        else filter_as_bf16<KS, 1, 2, DENSE>(g, smem, split, first_query);
        return;
    }
    for (int64_t q = first_query; q < first_query + kStatQueries && q < g.nq; q += kStatQueries / 2) {
        __syncthreads();                       // (the first half's last tile has been read)
        filter_as_bf16<KS, 2, 2, DENSE>(g, smem, split, q);
    }
}

// LDS of the general kernel, in bytes: vectors, queries, norms (two of each), thresholds
template <typename Elem>
struct GeneralLds {
    static constexpr int kQueries = 2 * (kGenRows / 32) * (sizeof(Elem) == 4 ? 2 : 1) * kFrag * 2;
    static constexpr int kNorms = kQueries + 2 * (kGenQueries / 32) * 2 * kFrag * 2;
    static constexpr int kFrom = kNorms + 2 * kGenRows * 4, kTotal = kFrom + kGenQueries * 4;
};

// Any dimension: both operands stream through LDS, 16 dimensions a step.  The workgroup's tile is 256 vectors x 128
// queries, a wavefront's 64 x 128 (128 accumulator registers); with two pieces on both sides a step is 24 matrix
// instructions (h.h, h.m, m.h) for 12 KB of LDS reads per wavefront.  A workgroup takes every splits-th tile of vectors;
// the steps of all its tiles are one sequence, so the next step's pieces are under way across tile borders too.
// Rows arrive as 64 bytes of floats per step, four lanes each, and are cut on their way into LDS (three instructions per
// element, a quarter of the matrix time and beside it); byte rows (more than 128 dimensions) as 16 bytes, one lane each.
template <typename Elem, bool DENSE>
__device__ __forceinline__ void filter_general(const BruteArgs& g, unsigned char* smem) {
    constexpr bool kFloats = sizeof(Elem) == 4;
    constexpr int XP = kFloats ? 2 : 1;                                        // pieces per value
    constexpr int kX = kGenRows / 32, kQ = kGenQueries / 32;                   // 32-row tiles of the workgroup's tile
    constexpr int kXPieces = kFloats ? 4 : 1, kQPieces = kQ * 2 * kFrag / 8 / kBfThreads;
    typedef GeneralLds<Elem> Lds;
    uint16_t* xs = reinterpret_cast<uint16_t*>(smem);                          // two of either, step by step in turn
    uint16_t* qs = reinterpret_cast<uint16_t*>(smem + Lds::kQueries);
    float* hs = reinterpret_cast<float*>(smem + Lds::kNorms);
    float* from = reinterpret_cast<float*>(smem + Lds::kFrom);
    constexpr int kXs = kX * XP * kFrag, kQs = kQ * 2 * kFrag;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int KS = g.KS, splits = g.splits;
    int split, group;
    place_of_workgroup(blockIdx.x, splits, (int)gridDim.x / splits, split, group);
    const int64_t q0 = (int64_t)group * kGenQueries;
    if (!DENSE && tid < kGenQueries) from[tid] = keep_from(g, g.keep, q0 + tid);      // (read after the first step's barrier)
    uint32_t count[kQ];
#pragma unroll
    for (int ct = 0; ct < kQ; ++ct) count[ct] = 0;
    const int ntile = (int)((g.chunk_rows + kGenRows - 1) / kGenRows);
    const u32x4* qf = reinterpret_cast<const u32x4*>(g.qfrag);
    constexpr int kTileQ = 2 * kFrag / 8;                                     // 16-byte pieces of a 32-query tile's step
    // the rows this thread brings 16 bytes of: (tid / 4) + 64 i, bytes 16 (tid % 4) of a step's 64; or row tid
    const int rl = kFloats ? tid >> 2 : tid, c4 = kFloats ? tid & 3 : 0;
    const uint64_t move = ((uint64_t)splits * kGenRows) % g.N * g.step % g.N;
    uint64_t id[kXPieces], hid;
#pragma unroll
    for (int i = 0; i < kXPieces; ++i) id[i] = ((g.chunk_pos + (uint64_t)split * kGenRows + rl + 64 * i) % g.N) * g.step % g.N;
    hid = ((g.chunk_pos + (uint64_t)split * kGenRows + tid) % g.N) * g.step % g.N;
    struct Step { u32x4 x[kXPieces], q[kQPieces]; };
    const bool centred = kFloats && g.use_centre[0] != 0u;
    int fks = 0;                               // the step fetched next, of the tile the ids stand for
    auto fetch = [&](Step& f) {                // (past the last tile: some vectors, unused; always loading keeps the pieces in registers)
        const int d = fks * 16 + 4 * c4;
        const bool in = d < g.D;               // D is a multiple of what a thread brings
#pragma unroll
        for (int i = 0; i < kXPieces; ++i) {
            const u32x4 zero = {0u, 0u, 0u, 0u};
            const u32x4 v = *reinterpret_cast<const u32x4*>(static_cast<const Elem*>(g.vectors) + id[i] * (uint64_t)g.D + (in ? d : 0));
            f.x[i] = in ? v : zero;
        }
#pragma unroll
        for (int i = 0; i < kQPieces; ++i) {
            const int e = i * kBfThreads + tid, ct = e / kTileQ;
            f.q[i] = qf[((size_t)(q0 / 32 + ct) * KS + fks) * kTileQ + e % kTileQ];
        }
        if (++fks == KS) {
            fks = 0;
#pragma unroll
            for (int i = 0; i < kXPieces; ++i) {
                id[i] += move;
                id[i] -= id[i] >= g.N ? g.N : 0;
            }
        }
    };
    v16f acc[2][kQ];
    auto step = [&](Step& f, int buf, int ks, float hx, float* hs) {
        const bool first = ks == 0;
        if constexpr (kFloats) {
            if (centred && ks * 16 + 4 * c4 < g.D) {           // (the zeros past the last dimension stay what they are)
                const u32x4 c = *reinterpret_cast<const u32x4*>(g.centre + ks * 16 + 4 * c4);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) f.x[i][j] = __float_as_uint(__uint_as_float(f.x[i][j]) - __uint_as_float(c[j]));
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {      // row r = rl + 64 i: 8 bytes of either piece
                const int r = rl + 64 * i;
                const float v0 = __uint_as_float(f.x[i][0]), v1 = __uint_as_float(f.x[i][1]), v2 = __uint_as_float(f.x[i][2]), v3 = __uint_as_float(f.x[i][3]);
                const uint32_t h0 = pack2(v0, v1), h1 = pack2(v2, v3);
                uint16_t* at = xs + buf * kXs + (r >> 5) * 2 * kFrag + (c4 >> 1) * 256 + (r & 31) * 8 + (c4 & 1) * 4;
                *reinterpret_cast<uint2*>(at) = make_uint2(h0, h1);
                *reinterpret_cast<uint2*>(at + kFrag) =
                    make_uint2(pack2(v0 - low_value(h0), v1 - high_value(h0)), pack2(v2 - low_value(h1), v3 - high_value(h1)));
            }
        } else {
            u32x4 w0, w1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t b = f.x[0][j];
                const uint32_t p0 = pack2((float)(b & 0xffu), (float)((b >> 8) & 0xffu)), p1 = pack2((float)((b >> 16) & 0xffu), (float)(b >> 24));
                if (j < 2) { w0[2 * j] = p0; w0[2 * j + 1] = p1; }
                else { w1[2 * j - 4] = p0; w1[2 * j - 3] = p1; }
            }
            u32x4* at = reinterpret_cast<u32x4*>(xs + buf * kXs) + (rl >> 5) * (kFrag / 8) + (rl & 31);
            at[0] = w0;
            at[32] = w1;
        }
#pragma unroll
        for (int i = 0; i < kQPieces; ++i) reinterpret_cast<u32x4*>(qs + buf * kQs)[i * kBfThreads + tid] = f.q[i];
        if (first) hs[tid] = -hx;
        __syncthreads();
        fetch(f);
        if (first) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                v16f c;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 h = *reinterpret_cast<const float4*>(&hs[wave * 64 + rt * 32 + 8 * i + 4 * (lane >> 5)]);
                    c[4 * i] = h.x; c[4 * i + 1] = h.y; c[4 * i + 2] = h.z; c[4 * i + 3] = h.w;
                }
#pragma unroll
                for (int ct = 0; ct < kQ; ++ct) acc[rt][ct] = c;
            }
        }
        bf16x8 a[2][XP];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int p = 0; p < XP; ++p)
                a[rt][p] = reinterpret_cast<const bf16x8*>(xs + buf * kXs)[((wave * 2 + rt) * XP + p) * (kFrag / 8) + lane];
#pragma unroll
        for (int ct = 0; ct < kQ; ++ct) {
            const bf16x8 h = reinterpret_cast<const bf16x8*>(qs + buf * kQs)[ct * kTileQ + lane];
            const bf16x8 m = reinterpret_cast<const bf16x8*>(qs + buf * kQs)[ct * kTileQ + kFrag / 8 + lane];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                acc[rt][ct] = mfma(a[rt][0], h, acc[rt][ct]);
                acc[rt][ct] = mfma(a[rt][0], m, acc[rt][ct]);
                if (XP > 1) acc[rt][ct] = mfma(a[rt][XP - 1], h, acc[rt][ct]);
            }
        }
    };
    // two steps are under way in registers: a step is 0.3 - 0.6 us of matrix work, less than a load takes
    Step f0, f1;
    fetch(f0);
    fetch(f1);
    int half = 0;
    bool odd = false;                          // which of the two holds the next step
    for (int t = split; t < ntile; t += splits, half ^= 1) {
        const float hx = (int64_t)t * kGenRows + tid < g.chunk_rows ? g.xhalf[hid] : __builtin_inff();    // such rows enter no list
        hid += move;
        hid -= hid >= g.N ? g.N : 0;
        int ks = 0;
        if (odd) {
            step(f1, 1, 0, hx, hs + half * kGenRows);
            ks = 1;
        }
        for (; ks + 1 < KS; ks += 2) {
            step(f0, 0, ks, hx, hs + half * kGenRows);
            step(f1, 1, ks + 1, hx, hs + half * kGenRows);
        }
        odd = ks < KS;
        if (odd) step(f0, 0, ks, hx, hs + half * kGenRows);
#pragma unroll
        for (int ct = 0; ct < kQ; ++ct) {
            const int64_t q = q0 + ct * 32 + (lane & 31);
            uint2* list = g.lists + ((size_t)q * g.segs + split * 8 + wave * 2 + (lane >> 5)) * g.seg_cap;
            float* dense = DENSE && q < g.nq ? g.dense + (size_t)q * kDense : nullptr;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
                take_tile<DENSE>(acc[rt][ct], DENSE ? 0.0f : from[ct * 32 + (lane & 31)], (uint32_t)t * kGenRows + wave * 64 + rt * 32 + 4 * (lane >> 5), dense, list, g.seg_cap, count[ct]);
        }
    }
    if (!DENSE) {
#pragma unroll
        for (int ct = 0; ct < kQ; ++ct)
            g.seg_count[(size_t)(q0 + ct * 32 + (lane & 31)) * g.segs + split * 8 + wave * 2 + (lane >> 5)] = count[ct];
    }
}

// Floats of a collection of up to kHalvesUpTo vectors: after the first chunk the products are of one piece of half precision on both
// sides, a third of the matrix work.  Eleven significant bits leave 2^-10 of a product, so more pairs pass: a window two to three times as
// wide where there are many dimensions (the additions of three products are allowed as much there), twelve times at 128.  A
// call keeps to bf16 if a norm is out of the range that is scaled to halves, or too many queries are crowded: they have more vectors
// of the first chunk in that window than they may (bf_select_kernel).  (The call as a whole: a group of 128 queries by itself takes the
// bf16 kernel as long as all of them, since its workgroups are the same few.  5,000 queries x 1M x 128 of which one in 20 groups of
// 256 kept to bf16 7.6 ms, all of them 5.6, by halves 3.5.)
// The workgroup's tile is 256 vectors x 256 queries, two times four wavefronts of 64 x 128; 32 dimensions a step, 16 matrix
// instructions a wavefront, so that a row is read by whole 128-byte lines.  Bound by LDS reads (half its cycles) and the barrier of a
// workgroup that has a compute unit to itself; workgroups of 128 queries, two per compute unit, read the vectors twice as often: 446 us
// for 777 queries x 150,001 x 960, with 16 dimensions a step 483.  LDS: the 16 bytes of a row's dimensions 8 j .. + 8 lie in slot
// row ^ 2 j (415 us without).
// The same, k = 10: the contraction after the first chunk 759 us by bf16 pieces, 404 by halves.
// What is kept gets exact fp32 distances, so that results are the same bits as by pieces (ten collections of 96 to 4,096 dimensions,
// 40,000 to 1M vectors; distances off from 64 bits by 1.6e-7 at most, the k nearest not at all, by either).
template <int QW>
struct HalvesLds {
    static constexpr int kVectors = kGenRows * 32 * 2, kQueries = QW * 128 * 32 * 2;       // a step's
    static constexpr int kQ = 2 * kVectors, kNorms = kQ + 2 * kQueries, kFrom = kNorms + 2 * kGenRows * 4, kScale = kFrom + QW * 128 * 4;
    static constexpr int kTotal = kScale + QW * 128 * 4;
};
__global__ __launch_bounds__(2 * kBfThreads, 2) void bf_halves_kernel(BruteArgs g) {
    constexpr int QW = kHalfQueries / kGenQueries;
    typedef HalvesLds<QW> Lds;
    __shared__ __align__(16) unsigned char smem[Lds::kTotal];
    constexpr int kQ = 4, kThreads = QW * kBfThreads, kXPieces = 8 / QW, kQPieces = 2;
    float* hs = reinterpret_cast<float*>(smem + Lds::kNorms);
    float* from = reinterpret_cast<float*>(smem + Lds::kFrom);
    float* scale = reinterpret_cast<float*>(smem + Lds::kScale);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, rw = wave & 3, qw = wave >> 2;
    if (!call_is_halves(g)) return;
    const int KS = g.KS, steps = (KS + 1) / 2, splits = g.splits_halves;
    int split, group;
    place_of_workgroup(blockIdx.x, splits, (int)gridDim.x / splits, split, group);
    const int64_t first_query = (int64_t)group * (QW * kGenQueries), q0 = first_query + qw * kGenQueries;
    const float xscale = half_scale(g.xhalf[g.N] + g.xhalf[g.N + 2]);
    if (tid < QW * kGenQueries) {                                              // (read after the first step's barrier)
        const bool have = first_query + tid < g.nq;
        scale[tid] = have ? xscale * half_scale(g.qnorm[first_query + tid]) : 1.0f;
        from[tid] = have ? keep_from(g, g.keep_halves, first_query + tid) * scale[tid] : __builtin_inff();
    }
    uint32_t count[kQ];
#pragma unroll
    for (int ct = 0; ct < kQ; ++ct) count[ct] = 0;
    const int ntile = (int)((g.chunk_rows + kGenRows - 1) / kGenRows);
    const u32x4* qf = reinterpret_cast<const u32x4*>(g.qhalf);
    const int last_tile = (int)((g.nq + 31) / 32) - 1;                         // (past it: its queries again, kept by nobody)
    // the rows this thread brings 16 bytes of: (tid / 8) + 32 QW i, bytes 16 (tid % 8) of a step's 128; row tid's norm
    const int rl = tid >> 3, c8 = tid & 7;
    const uint32_t N = (uint32_t)g.N, move = (uint32_t)(((uint64_t)splits * kGenRows) % g.N * g.step % g.N);      // (N is at most kHalvesUpTo)
    uint32_t id[kXPieces], hid;
#pragma unroll
    for (int i = 0; i < kXPieces; ++i) id[i] = (uint32_t)(((g.chunk_pos + (uint64_t)split * kGenRows + rl + 32 * QW * i) % g.N) * g.step % g.N);
    hid = (uint32_t)(((g.chunk_pos + (uint64_t)split * kGenRows + tid) % g.N) * g.step % g.N);
    auto advance = [&](uint32_t& at) {
        at += move;
        at -= at >= N ? N : 0u;
    };
    const bool centred = g.use_centre[0] != 0u;
    struct Step { u32x4 x[kXPieces], q[kQPieces]; };
    int fks = 0;                               // the step fetched next, of the tile the ids stand for
    auto fetch = [&](Step& f) {                // (past the last tile: some vectors, unused; always loading keeps the pieces in registers)
        const int d = fks * 32 + 4 * c8;
        const bool in = d < g.D;
#pragma unroll
        for (int i = 0; i < kXPieces; ++i) {
            const u32x4 zero = {0u, 0u, 0u, 0u};
            const u32x4 v = *reinterpret_cast<const u32x4*>(static_cast<const float*>(g.vectors) + id[i] * (uint64_t)g.D + (in ? d : 0));
            f.x[i] = in ? v : zero;
        }
#pragma unroll
        for (int i = 0; i < kQPieces; ++i) {   // (an odd last step: the queries' last sixteen dimensions against zeros)
            const int e = i * kThreads + tid, qt = min((int)(first_query / 32) + e / 128, last_tile), ks = min(2 * fks + (e / 64) % 2, KS - 1);
            f.q[i] = qf[((size_t)qt * KS + ks) * (kFrag / 8) + e % 64];
        }
        if (++fks == steps) {
            fks = 0;
#pragma unroll
            for (int i = 0; i < kXPieces; ++i) advance(id[i]);
        }
    };
    v16f acc[2][kQ];
    int t = split, ks = 0, half = 0;
    float hx = 0.0f;
    auto step = [&](Step& f, int buf) {        // false: that was the last
        uint16_t* xs = reinterpret_cast<uint16_t*>(smem + buf * Lds::kVectors);
        u32x4* qs = reinterpret_cast<u32x4*>(smem + Lds::kQ + buf * Lds::kQueries);
        float* norms = hs + half * kGenRows;
        if (ks == 0 && tid < kGenRows) {
            hx = (int64_t)t * kGenRows + tid < g.chunk_rows ? g.xhalf_halves[hid] : __builtin_inff();     // such rows enter no list
            advance(hid);
        }
        const int d = ks * 32 + 4 * c8;
        u32x4 c = {0u, 0u, 0u, 0u};
        if (centred && d < g.D) c = *reinterpret_cast<const u32x4*>(g.centre + d);         // (the zeros past the last dimension stay what they are)
        float less[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) less[j] = -__uint_as_float(c[j]) * xscale;             // (a power of two: rounded as before scaling)
#pragma unroll
        for (int i = 0; i < kXPieces; ++i) {
            const int r = rl + 32 * QW * i;
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = fmaf(__uint_as_float(f.x[i][j]), xscale, less[j]);
            *reinterpret_cast<uint2*>(xs + ((r >> 5) * 2 + (c8 >> 2)) * kFrag + ((c8 >> 1) & 1) * 256 + ((r & 31) ^ (c8 & 6)) * 8 + (c8 & 1) * 4) =
                make_uint2(pack2_half(v[0], v[1]), pack2_half(v[2], v[3]));
        }
#pragma unroll
        for (int i = 0; i < kQPieces; ++i) qs[i * kThreads + tid] = f.q[i];
        if (ks == 0 && tid < kGenRows) norms[tid] = -hx;
        __syncthreads();
        fetch(f);
        if (ks == 0) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                v16f start;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 h = *reinterpret_cast<const float4*>(&norms[rw * 64 + rt * 32 + 8 * i + 4 * (lane >> 5)]);
                    start[4 * i] = h.x; start[4 * i + 1] = h.y; start[4 * i + 2] = h.z; start[4 * i + 3] = h.w;
                }
#pragma unroll
                for (int ct = 0; ct < kQ; ++ct) {
                    const float own = scale[qw * kGenQueries + ct * 32 + (lane & 31)];
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[rt][ct][r] = start[r] * own;
                }
            }
        }
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            bf16x8 a[2];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) a[rt] = reinterpret_cast<const bf16x8*>(xs)[((rw * 2 + rt) * 2 + sub) * (kFrag / 8) + (lane ^ (4 * sub + 2 * (lane >> 5)))];
#pragma unroll
            for (int ct = 0; ct < kQ; ++ct) {
                const bf16x8 h = reinterpret_cast<const bf16x8*>(qs)[((qw * kQ + ct) * 2 + sub) * (kFrag / 8) + lane];
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) acc[rt][ct] = mfma_half(a[rt], h, acc[rt][ct]);
            }
        }
        if (++ks < steps) return true;
        ks = 0;
#pragma unroll
        for (int ct = 0; ct < kQ; ++ct) {
            const int at = qw * kGenQueries + ct * 32 + (lane & 31);
            const int64_t q = first_query + at;
            uint2* list = g.lists + ((size_t)q * g.segs + split * 8 + rw * 2 + (lane >> 5)) * g.seg_cap;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
                take_tile<false>(acc[rt][ct], from[at], (uint32_t)t * kGenRows + rw * 64 + rt * 32 + 4 * (lane >> 5), nullptr, list, g.seg_cap, count[ct],
                                 1.0f / scale[at]);
        }
        t += splits;
        half ^= 1;
        return t < ntile;
    };
    // two steps are under way in registers
    if (t < ntile) {
        Step f0, f1;
        fetch(f0);
        fetch(f1);
        while (step(f0, 0) && step(f1, 1)) {}
    }
#pragma unroll
    for (int ct = 0; ct < kQ; ++ct)
        if (q0 + ct * 32 + (lane & 31) < g.nq) {
            uint32_t* counts = g.seg_count + (size_t)(q0 + ct * 32 + (lane & 31)) * g.segs + rw * 2 + (lane >> 5);
            counts[split * 8] = count[ct];
            for (int s = split + splits; s < g.splits; s += splits) counts[s * 8] = 0u;    // lists that only the bf16 kernel fills
        }
}

template <typename Elem, bool DENSE>
__global__ __launch_bounds__(kBfThreads, 2) void bf_filter_kernel(BruteArgs g) {
    __shared__ __align__(16) unsigned char smem[GeneralLds<Elem>::kTotal];
    if constexpr (sizeof(Elem) == 4 && !DENSE)
        if (call_is_halves(g)) return;                                         // bf_halves_kernel has it
    filter_general<Elem, DENSE>(g, smem);
}

constexpr int kSelectBins = 1024;

constexpr int kBest = 2048;            // entries kept of a query between chunks: the k best and what may tie with them

// One workgroup per query: what is kept of the list so far and of the chunk's new pairs (dense: of the first chunk's
// values); after the last chunk the exact distances of the kept vectors and the k best of them.
// Entries: bits of s~ << 32 | place in the database order.  (Bins are equal pieces of the value range, not of the bit
// patterns: s~ changes sign, and most of the patterns between its smallest and largest value are next to zero.)
template <typename Elem>
__global__ __launch_bounds__(kBfThreads) void bf_select_kernel(BruteArgs g, int dense, int last, int rank, uint32_t few) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned long long* keys = reinterpret_cast<unsigned long long*>(smem);    // kDense
    __shared__ uint32_t hist[kSelectBins];
    __shared__ uint32_t part[kBfThreads / kWave];
    __shared__ float bounds[2 * kBfThreads / kWave];
    __shared__ uint32_t misc[8];                    // 2 chosen bin, 3 entries kept, 4 overflow, 5, 6 entries before and up to its end
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, k = g.k;
    const int64_t q = blockIdx.x;
    if (g.flagged[q]) return;
    unsigned long long* best = g.best + (size_t)q * kBest;
    if (tid == 0) {
        misc[3] = misc[4] = 0u;
    }
    for (int e = tid; e < kSelectBins; e += kBfThreads) hist[e] = 0u;
    __syncthreads();

    // ---- everything into LDS -----------------------------------------------------------------------------------
    int n;
    if (dense) {
        n = (int)g.chunk_rows;
        const float* row = g.dense + (size_t)q * kDense;
        constexpr int kPer = kDense / 4 / kBfThreads;                            // 16 bytes at a time, all asked for at once
        float4 v[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) v[u] = reinterpret_cast<const float4*>(row)[4 * (tid + u * kBfThreads) < n ? tid + u * kBfThreads : 0];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = 4 * (tid + u * kBfThreads);
            const float w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (e + c < n) keys[e + c] = ((unsigned long long)__float_as_uint(w[c]) << 32) | (uint32_t)(e + c);
        }
    } else {
        const int nb = (int)g.best_count[q];
        for (int e = tid; e < nb; e += kBfThreads) keys[e] = best[e];
        n = nb;
        for (int s0 = 0; s0 < g.segs; s0 += kBfThreads) {
            const int s = s0 + tid;
            const uint32_t c = s < g.segs ? g.seg_count[(size_t)q * g.segs + s] : 0u;
            uint32_t total;
            const uint32_t at = (uint32_t)n + block_exclusive_sum(min(c, (uint32_t)kDense), part, total);
            if (c > (uint32_t)g.seg_cap || (uint32_t)n + total > (uint32_t)kDense) misc[4] = 1u;
            __syncthreads();                         // (its next change comes after a barrier that everyone reaches past this test)
            if (misc[4]) break;
            const uint2* list = g.lists + ((size_t)q * g.segs + s) * g.seg_cap;
            for (uint32_t i = 0; i < c; ++i)
                keys[at + i] = ((unsigned long long)list[i].y << 32) | (uint32_t)(g.chunk_pos + list[i].x);
            n += (int)total;
        }
    }
    __syncthreads();
    const float qn = g.qnorm[q];
    auto give_up = [&]() {                           // to the exact scan
        if (tid == 0) {
            g.flagged[q] = 1u;
            g.todo[atomicAdd(&g.control[kBfTodo], 1u)] = (uint32_t)q;
        }
    };
    // the same for the whole workgroup; with these norms all values are finite
    if (misc[4] || !(qn < 1e18f) || !(g.xhalf[g.N] < 1e18f)) {
        give_up();
        return;
    }
    const float before = dense ? __builtin_inff() : g.edge[q];                  // the bound so far: the list holds all up to it, and more
    // a guess was too small: fewer than k vectors are up to it
    if (last && n < k) {
        give_up();
        return;
    }
    // ---- an upper bound of the rank-th smallest: the end of its bin ------------------------------------------------
    // One histogram over the values' range; where a few long vectors stretch the range, so that the bin of the k-th holds many
    // more than `few` up to its end, its entries get a histogram of their own, and so on.  Bit u of `members`: entry tid + u * 256 is
    // among those that are divided.
    auto value = [&](int e) { return __uint_as_float((uint32_t)(keys[e] >> 32)); };
    static_assert(kDense <= 32 * kBfThreads, "a bit per entry");
    uint32_t members = 0xffffffffu, below = 0u;
    float edge = before, least = 0.0f;
    auto divide = [&](auto all) {                    // one histogram; false: the bin's entries are to be divided
        constexpr bool ALL = decltype(all)::value;   // every entry is a member
        float lo = __builtin_inff(), hi = -__builtin_inff();
        for (int e = tid, u = 0; e < n; e += kBfThreads, ++u)
            if (ALL || (members >> u & 1u)) {
                lo = fminf(lo, value(e));
                hi = fmaxf(hi, value(e));
            }
        for (int off = 32; off > 0; off >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, off, kWave));
            hi = fmaxf(hi, __shfl_xor(hi, off, kWave));
        }
        if (lane == 0) {
            bounds[2 * wave] = lo;
            bounds[2 * wave + 1] = hi;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kBfThreads / kWave; ++w) {
            lo = fminf(lo, bounds[2 * w]);
            hi = fmaxf(hi, bounds[2 * w + 1]);
        }
        edge = hi;
        if (ALL) least = lo;
        if (!(hi - lo > 1e-30f)) return true;        // equal, or next to it
        const float scale = (float)kSelectBins / (hi - lo);
        auto bin_of = [&](float v) { return (int)fminf((v - lo) * scale, (float)(kSelectBins - 1)); };
        for (int e = tid, u = 0; e < n; e += kBfThreads, ++u)
            if (ALL || (members >> u & 1u)) atomicAdd(&hist[bin_of(value(e))], 1u);
        __syncthreads();
        {
            constexpr int bpt = kSelectBins / kBfThreads;
            uint32_t h[bpt], sum = 0, total;
#pragma unroll
            for (int j = 0; j < bpt; ++j) {
                sum += h[j] = hist[tid * bpt + j];
                hist[tid * bpt + j] = 0u;
            }
            uint32_t c = below + block_exclusive_sum(sum, part, total);
#pragma unroll
            for (int j = 0; j < bpt; ++j) {
                if (c < (uint32_t)rank && (uint32_t)rank <= c + h[j]) {
                    misc[2] = (uint32_t)(tid * bpt + j);
                    misc[5] = c;
                    misc[6] = c + h[j];
                }
                c += h[j];
            }
        }
        __syncthreads();
        // the end of the bin, a little behind it for the rounding of the bin numbers
        const int bin = (int)misc[2];
        below = misc[5];
        edge = fminf(hi, lo + (float)(bin + 1) / scale * 1.000002f + 4e-7f * fabsf(lo));
        if (misc[6] <= few) return true;
        for (int e = tid, u = 0; e < n; e += kBfThreads, ++u)
            if (bin_of(value(e)) != bin) members &= ~(1u << u);
        return false;
    };
    if (n >= rank) {                                 // (else the list is as it was)
        bool done = divide(std::true_type{});
        for (int level = 0; level < 3 && !done; ++level) done = divide(std::false_type{});
    }
    if (edge > before) {                             // the bin's end, or the rank-th itself
        edge = before;
        if (last) {
            __syncthreads();                         // (misc[2] has been read)
            if (tid == 0) misc[2] = 0u;
            __syncthreads();
            uint32_t up_to = 0;
            for (int e = tid; e < n; e += kBfThreads) up_to += value(e) <= before ? 1u : 0u;
            atomicAdd(&misc[2], up_to);
            __syncthreads();
            if (misc[2] < (uint32_t)k) {             // the guess was too small
                give_up();
                return;
            }
        }
    }
    // (values of bytes against bytes are exact: half squared distances rounded down, but for a term of the query)
    const bool exact = sizeof(Elem) == 1 && g.qbytes && group_is_bytes(g, (int)(q / kStatQueries));
    float keep = exact ? edge : keep_up_to(g, g.err, qn, g.qshift[q], edge);
    if (!last && tid == 0) g.keep[q] = keep;
    if (sizeof(Elem) == 4 && g.qhalf && !(dense && last)) {
        const float wide = keep_up_to(g, g.err_half, qn, g.qshift[q], edge);
        if (!last && tid == 0) g.keep_halves[q] = wide;
        if (!dense) {
            if (call_is_halves(g)) keep = wide;
        } else if (g.second[q / 32] & kNoHalves) {
            if (tid == 0) atomicOr(&g.control[kBfCrowded], kHalvesOff);
        } else {                                     // (this chunk's values are those of bf16 pieces)
            // Is there room for what the halves' window lets pass?  In the next chunk as much as in this one, in proportion; in the
            // end what is in the window of the k nearest: as large a share of all vectors as of these, if they are crowded there; where
            // the values thin out towards the nearest, k times what a window from the nearest of these holds.
            auto count_up_to = [&](float bound) {    // (to misc[2])
                __syncthreads();                     // (misc[2] has been read)
                if (tid == 0) misc[2] = 0u;
                __syncthreads();
                uint32_t up_to = 0;
                for (int e = tid; e < n; e += kBfThreads) up_to += value(e) <= bound ? 1u : 0u;
                atomicAdd(&misc[2], up_to);
                __syncthreads();
                return misc[2];
            };
            const uint32_t up_to = count_up_to(wide);
            const float share = (float)g.N / (float)kDense;
            bool crowded = (int)up_to > g.crowded_next;
            const bool full = up_to > (uint32_t)kBest;                         // (not even now: this query's list is one for bf16)
            if (!crowded && share * (float)up_to > (float)kBest)               // (the same for the whole workgroup)
                crowded = fmaxf(share, (float)k) * (float)count_up_to(keep_up_to(g, g.err_half, qn, g.qshift[q], least)) > (float)kBest;
            if (!full) keep = wide;
            if (tid == 0 && full) atomicOr(&g.control[kBfCrowded], kHalvesOff);
            else if (tid == 0 && crowded) atomicAdd(&g.control[kBfCrowded], 1u);
        }
    }
    // ---- keep what can still be among the k nearest ---------------------------------------------------------------
    for (int e0 = 0; e0 < n; e0 += kBfThreads) {     // in place: entry e moves to a place <= e that has been read
        const int e = e0 + tid;
        const unsigned long long key = e < n ? keys[e] : ~0ull;
        const bool take = e < n && __uint_as_float((uint32_t)(key >> 32)) <= keep;
        const unsigned long long m = __ballot(take);
        uint32_t at = 0;
        __syncthreads();                             // this round's entries have been read
        if (lane == 0 && m) at = atomicAdd(&misc[3], (uint32_t)__popcll(m));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (take) keys[at] = key;
    }
    __syncthreads();
    n = (int)misc[3];
    if (n > kBest) {
        give_up();
        return;
    }
    if (!last) {
        for (int e = tid; e < n; e += kBfThreads) best[e] = keys[e];
        if (tid == 0) {
            g.best_count[q] = (uint32_t)n;
            g.edge[q] = edge;
        }
        return;
    }
    // ---- exact distances of the kept vectors, the k best by (distance, id) ------------------------------------------
    float4* sy = reinterpret_cast<float4*>(smem + sizeof(unsigned long long) * kDense);        // D floats
    const int D = g.D;
    for (int c4 = tid; c4 < D / 4; c4 += kBfThreads) sy[c4] = reinterpret_cast<const float4*>(g.queries + (size_t)q * D)[c4];
    const int npad = next_pow2(n) < 64 ? 64 : next_pow2(n);
    for (int e = n + tid; e < npad; e += kBfThreads) keys[e] = ~0ull;
    __syncthreads();
    const int lpr = lanes_per_row(D / Piece<Elem>::kElems);
    const int per_wave = kWave / lpr, sub = lane / lpr, l = lane & (lpr - 1);
    // (four rows on their way, as in the exact re-ranking; a row past the end is the group's first once more)
    constexpr int kRows = 4;
    const int npieces = D / Piece<Elem>::kElems, rows_per_iter = per_wave * (kBfThreads / kWave);
    const float* y = reinterpret_cast<const float*>(sy);
    for (int e0 = wave * per_wave + sub; e0 < n; e0 += kRows * rows_per_iter) {
        const uint4* x[kRows];
        uint32_t id[kRows];
        float acc[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int e = e0 + u * rows_per_iter;
            const uint32_t place = (uint32_t)keys[e < n ? e : e0];
            id[u] = (uint32_t)((uint64_t)place * g.step % g.N);
            x[u] = reinterpret_cast<const uint4*>(static_cast<const Elem*>(g.vectors) + (size_t)id[u] * D);
            acc[u] = 0.0f;
        }
        for (int piece = l; piece < npieces; piece += lpr) {
            uint4 raw[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) raw[u] = x[u][piece];
#pragma unroll
            for (int u = 0; u < kRows; ++u) acc[u] = Piece<Elem>::add(raw[u], piece, y, acc[u]);
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            for (int off = 1; off < lpr; off <<= 1) acc[u] += __shfl_xor(acc[u], off, kWave);
            const int e = e0 + u * rows_per_iter;
            if (e < n && l == 0) keys[e] = ((unsigned long long)mono_key(acc[u]) << 32) | id[u];
        }
    }
    if (npad <= 4 * kBfThreads) block_sort_lds<4>(keys, npad, tid, kBfThreads);
    else block_sort_lds<8>(keys, npad, tid, kBfThreads);
    for (int e = tid; e < k; e += kBfThreads) {
        const unsigned long long key = keys[e];
        g.out_ids[(size_t)q * k + e] = (int64_t)(uint32_t)key;
        g.out_dists[(size_t)q * k + e] = mono_inv((uint32_t)(key >> 32));
    }
}

// The queries the filter gave up on: exact distances to every vector, what beats the k-th best so far is kept in LDS and
// the k best are selected again whenever that may fill.  A workgroup has QB queries, which share the rows it reads (two at a
// time in registers: each of the queries' values in LDS is read once for both), and one of `splits` parts of the database, as many
// as give every workgroup of the launch work; the workgroup that ends the last of several parts joins their results.
// 2,000 queries that all tie, 1M x 128 bytes: 20.6 ms (one workgroup per query, a row read for one query: 47); one such query:
// 0.36 ms (20.7).
constexpr int kScanQueries = 4;
constexpr int kScanSplits = 256;       // parts of the database at most
constexpr int kScanKeys = 1024;        // entries a workgroup holds per query: the k best and what is pending
constexpr int kScanStep = 512;         // rows between two looks at the number of pending entries, at most

constexpr size_t scan_lds(int queries, int D) { return (size_t)queries * (sizeof(unsigned long long) * kScanKeys + sizeof(float) * D) + 64; }

__device__ __forceinline__ uint32_t scan_splits(uint32_t ntodo, uint32_t queries, uint32_t grid, uint64_t N) {
    const uint32_t blocks = (ntodo + queries - 1) / queries;
    const uint32_t rows = (uint32_t)((N + kScanStep - 1) / kScanStep);
    return max(1u, min(min(grid / blocks, (uint32_t)kScanSplits), rows));
}

// The k best of the parts of a scanned query, by one workgroup; keys: kScanKeys entries.
__device__ __forceinline__ void merge_parts(const BruteArgs& g, uint32_t at, int splits, unsigned long long* keys, uint32_t* pending) {
    constexpr int kStep = kScanKeys / 2;
    const int tid = threadIdx.x, k = g.k, total = splits * k;
    const unsigned long long* parts = g.parts + (size_t)at * total;
    for (int e = tid; e < k; e += kBfThreads) keys[e] = ~0ull;
    if (tid == 0) *pending = 0u;
    __syncthreads();
    unsigned long long tau = ~0ull;
    for (int e0 = 0; e0 < total; e0 += kStep) {
#pragma unroll
        for (int u = 0; u < kStep / kBfThreads; ++u) {
            const int e = e0 + u * kBfThreads + tid;
            const unsigned long long key = e < total ? parts[e] : ~0ull;
            if (key < tau) keys[k + atomicAdd(pending, 1u)] = key;
        }
        __syncthreads();
        const uint32_t np = *pending;
        __syncthreads();
        if (np + (uint32_t)kStep > (uint32_t)(kScanKeys - k) || e0 + kStep >= total) {
            const int n = k + (int)np, npad = next_pow2(n) < 64 ? 64 : next_pow2(n);
            for (int e = n + tid; e < npad; e += kBfThreads) keys[e] = ~0ull;
            if (tid == 0) *pending = 0u;
            block_sort_lds<4>(keys, npad, tid, kBfThreads);
            tau = keys[k - 1];
            __syncthreads();
        }
    }
    const size_t q = g.todo[at];
    for (int e = tid; e < k; e += kBfThreads) {
        const unsigned long long key = keys[e];
        g.out_ids[q * k + e] = key == ~0ull ? -1 : (int64_t)(uint32_t)key;
        g.out_dists[q * k + e] = key == ~0ull ? __builtin_inff() : mono_inv((uint32_t)(key >> 32));
    }
    __syncthreads();
}

template <typename Elem, int QB>
__global__ __launch_bounds__(kBfThreads, 4) void bf_scan_kernel(BruteArgs g) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned long long* keys = reinterpret_cast<unsigned long long*>(smem);    // [QB][kScanKeys]
    float* sy = reinterpret_cast<float*>(smem + sizeof(unsigned long long) * QB * kScanKeys);      // [QB][D]
    __shared__ uint32_t pending[QB], parts_done;
    constexpr int kRows = 2;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, k = g.k, D = g.D;
    const uint32_t ntodo = g.control[kBfTodo];
    if (ntodo == 0) return;
    const int npieces = D / Piece<Elem>::kElems, lpr = lanes_per_row(npieces);
    const int per_wave = kWave / lpr, sub = lane / lpr, l = lane & (lpr - 1);
    const int per_iter = kRows * per_wave * (kBfThreads / kWave), iters = kScanStep / per_iter;      // 4 .. 512 rows, 1 .. 64 of them
    const uint32_t splits = scan_splits(ntodo, QB, gridDim.x, g.N), blocks = (ntodo + QB - 1) / QB;
    const Elem* X = reinterpret_cast<const Elem*>(g.vectors);
    for (uint32_t item = blockIdx.x; item < blocks * splits; item += gridDim.x) {
        const uint32_t first = item / splits * QB, split = item % splits;
        const int64_t x_end = (int64_t)(g.N * (split + 1) / splits);
        __syncthreads();
        for (int e = tid; e < QB * (D / 4); e += kBfThreads) {
            const int j = e / (D / 4), c4 = e - j * (D / 4);
            const int64_t q = g.todo[min(first + (uint32_t)j, ntodo - 1)];     // (past the last query: it once more)
            reinterpret_cast<float4*>(sy)[e] = reinterpret_cast<const float4*>(g.queries + (size_t)q * D)[c4];
        }
        for (int j = 0; j < QB; ++j)
            for (int e = tid; e < k; e += kBfThreads) keys[j * kScanKeys + e] = ~0ull;
        if (tid < QB) pending[tid] = 0u;
        __syncthreads();
        uint32_t tau[QB];
#pragma unroll
        for (int j = 0; j < QB; ++j) tau[j] = 0xffffffffu;
        for (int64_t x0 = (int64_t)(g.N * split / splits); x0 < x_end; x0 += (int64_t)iters * per_iter) {
            for (int it = 0; it < iters; ++it) {
                int64_t row[kRows];
                const Elem* x[kRows];
                float acc[kRows][QB];
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    row[r] = x0 + it * per_iter + (wave * kRows + r) * per_wave + sub;
                    x[r] = X + (size_t)(row[r] < x_end ? row[r] : x_end - 1) * D;
#pragma unroll
                    for (int j = 0; j < QB; ++j) acc[r][j] = 0.0f;
                }
                for (int piece = l; piece < npieces; piece += lpr) {
                    uint4 raw[kRows];
#pragma unroll
                    for (int r = 0; r < kRows; ++r) raw[r] = reinterpret_cast<const uint4*>(x[r])[piece];
#pragma unroll
                    for (int j = 0; j < QB; ++j)
#pragma unroll
                        for (int r = 0; r < kRows; ++r) acc[r][j] = Piece<Elem>::add(raw[r], piece, sy + j * D, acc[r][j]);
                }
                for (int off = 1; off < lpr; off <<= 1)
#pragma unroll
                    for (int r = 0; r < kRows; ++r)
#pragma unroll
                        for (int j = 0; j < QB; ++j) acc[r][j] += __shfl_xor(acc[r][j], off, kWave);
                // vectors come in id order: an equal distance that arrives later has the larger id and never wins
#pragma unroll
                for (int r = 0; r < kRows; ++r)
#pragma unroll
                    for (int j = 0; j < QB; ++j) {
                        const uint32_t kb = mono_key(acc[r][j]);
                        if (l == 0 && row[r] < x_end && kb < tau[j])
                            keys[j * kScanKeys + k + atomicAdd(&pending[j], 1u)] = ((unsigned long long)kb << 32) | (uint32_t)row[r];
                    }
            }
            __syncthreads();
            uint32_t np[QB];
#pragma unroll
            for (int j = 0; j < QB; ++j) np[j] = pending[j];
            __syncthreads();
            const bool last = x0 + (int64_t)iters * per_iter >= x_end;
#pragma unroll
            for (int j = 0; j < QB; ++j) {
                if (np[j] + (uint32_t)kScanStep <= (uint32_t)(kScanKeys - k) && !last) continue;
                unsigned long long* own = keys + j * kScanKeys;
                const int n = k + (int)np[j], npad = next_pow2(n) < 64 ? 64 : next_pow2(n);
                for (int e = n + tid; e < npad; e += kBfThreads) own[e] = ~0ull;
                if (tid == 0) pending[j] = 0u;
                block_sort_lds<4>(own, npad, tid, kBfThreads);
                tau[j] = (uint32_t)(own[k - 1] >> 32);
                __syncthreads();
            }
        }
        for (int j = 0; j < QB; ++j) {
            const uint32_t at = first + (uint32_t)j;
            if (at >= ntodo) break;
            const size_t q = g.todo[at];
            for (int e = tid; e < k; e += kBfThreads) {
                const unsigned long long key = keys[j * kScanKeys + e];
                if (splits > 1) {
                    g.parts[((size_t)at * splits + split) * k + e] = key;
                } else {
                    g.out_ids[q * k + e] = key == ~0ull ? -1 : (int64_t)(uint32_t)key;
                    g.out_dists[q * k + e] = key == ~0ull ? __builtin_inff() : mono_inv((uint32_t)(key >> 32));
                }
            }
        }
        if (splits > 1) {                              // the workgroup that ends the last part of these queries joins them
            __threadfence();
            __syncthreads();
            if (tid == 0) parts_done = atomicAdd(&g.scan_done[item / splits], 1u);
            __syncthreads();
            if (parts_done == splits - 1u) {
                __threadfence();
                for (uint32_t at = first; at < first + (uint32_t)QB && at < ntodo; ++at) merge_parts(g, at, (int)splits, keys, pending);
            }
        }
    }
}

uint64_t gcd_u64(uint64_t a, uint64_t b) {
    while (b) {
        const uint64_t t = a % b;
        a = b;
        b = t;
    }
    return a;
}

// where the centre (bytes: the whole half norms of the vectors less 128) stands behind the N half norms, the largest norm, the word that says whether it is subtracted, and its norm where
// it is not: at a 16-byte boundary
size_t centre_at(uint64_t N) { return (size_t)(N + 6) / 4 * 4; }

// floats: what values of products of halves start from
size_t halves_at(uint64_t N, int D) { return centre_at(N) + (size_t)(D + 3) / 4 * 4; }

int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// How many of the k nearest of N vectors the first `pos` places of the database order hold, hardly ever exceeded (less than once in
// 10^8 for vectors in any order that the golden ratio knows nothing of).
int rank_at(int k, double pos, double N) {
    const double p = pos < N ? pos / N : 1.0, mean = k * p;
    const double most = mean + 6.0 * std::sqrt(mean * (1.0 - p)) + 4.0;
    return most < k ? (int)most : k;
}

// Floats: the largest collection that is filtered by halves.  Where more vectors than the kept lists hold (kBest) are in their window,
// some have to show in the first chunk: eight of them in the mean.
constexpr uint64_t kHalvesUpTo = (uint64_t)kBest * kDense / 8;

// How one call is cut: sizes of the workspace's pieces and the launch shapes.
struct Plan {
    bool stationary, halves;
    int KS;
    int64_t batch, batch_pad;        // queries at a time, padded to whole workgroup tiles
    int groups, splits, splits_halves, segs, seg_cap;
    double growth;                   // chunks and what was there before them
    int hits;                        // pairs that pass in a chunk
    int scan_queries, scan_grid;     // of the exact scan: queries and workgroups
};

Plan make_plan(int64_t nq, uint64_t N, int D, int elem_bytes, int k) {
    Plan p;
    p.KS = (D + 15) / 16;
    p.stationary = elem_bytes == 1 && p.KS <= 8;
    if (p.stationary && p.KS != 6) p.KS = 8;                        // compiled for 96 and 128 dimensions
    const int tile = p.stationary ? kStatQueries : kGenQueries;
    p.batch = nq < 16384 ? nq : 16384;
    p.batch_pad = round_up(p.batch, tile);
    // Halves need the queries a second time and a look at the first chunk, about 6 us: not for what takes less than a few
    // times that.  (Up to 128 queries the workgroup's second half would idle.)  A step is 32 dimensions, one of 16 would be half
    // padding: 1,000 queries x 1M x 16, k = 100: 262 us by bf16 pieces, 292 by halves; x 64 494 and 373.
    p.halves = elem_bytes == 4 && D > 32 && N >= 8 * kDense && N <= kHalvesUpTo && p.batch > kGenQueries && (double)p.batch_pad * (double)N * D > 6e9;
    p.groups = (int)(p.batch_pad / tile);
    // as many workgroups as are resident at once (two per compute unit): no second round of a few
    const int slots = 512;
    p.splits = p.groups >= slots ? 1 : slots / p.groups;
    if (p.splits > 8) p.splits -= p.splits % 8;
    p.splits_halves = std::max(1, std::min(p.splits, 256 / ((p.groups + 1) / 2)));             // (one workgroup of bf_halves_kernel per compute unit)
    if (p.splits_halves > 8) p.splits_halves -= p.splits_halves % 8;
    p.segs = p.splits * (p.stationary ? 2 : 8);
    // As many chunks, each larger by the same factor, as take the least time: a chunk costs a launch of either kernel and a
    // look at every query's list, a pair that passes some hundred cycles of its wavefront, which takes 128 queries.  Bounded by
    // the select workgroup's LDS (the pairs, twice the expected number, and the list kept so far; halves let through twice as many).
    const double room = p.halves ? 800.0 : 1600.0;
    p.growth = 2.0;
    p.hits = k;
    double least = 1e30;
    const double waves = 512.0 * (p.stationary && p.batch < 384 ? (double)((p.batch + 127) / 128) : 4.0);
    for (int chunks = 1; chunks <= 16 && N > kDense; ++chunks) {
        const double growth = std::pow((double)N / kDense, 1.0 / chunks) * 1.001;
        double time = 0.0, most = 0.0, pos = kDense;
        for (int c = 0; c < chunks; ++c, pos *= growth) {
            const double hits = rank_at(k, pos, (double)N) * (growth - 1.0);
            time += 10.0 + 0.005 * (double)p.batch + 0.2 * hits * (double)p.batch / waves;
            most = hits > most ? hits : most;
        }
        if (time < least && (most <= room || growth <= 2.0)) {
            least = time;
            p.growth = growth;
            p.hits = (int)most + 1;
        }
    }
    // room for the pairs that pass and for the ties that may be kept
    p.seg_cap = 4 * ((p.hits + p.segs - 1) / p.segs) + 16 + kBest / p.segs;
    p.scan_queries = scan_lds(kScanQueries, D) <= 63 * 1024 ? kScanQueries : 1;      // (64 KB less what the kernel has itself)
    const int64_t most_items = (p.batch + p.scan_queries - 1) / p.scan_queries * kScanSplits;
    p.scan_grid = (int)(most_items < 1024 ? most_items : 1024);
    return p;
}

struct Carver {
    unsigned char* base;
    size_t used = 0;
    template <typename T>
    T* take(size_t count) {
        T* p = base ? reinterpret_cast<T*>(base + used) : nullptr;
        used += (count * sizeof(T) + 255) / 256 * 256;
        return p;
    }
};

size_t carve(const Plan& p, int k, unsigned char* base, BruteArgs* a) {
    Carver c{base};
    BruteArgs v = {};
    v.control = c.take<uint32_t>(kBfControl);
    v.flagged = c.take<uint32_t>(p.batch_pad);
    v.second = c.take<uint32_t>(p.batch_pad / 32);
    v.todo = c.take<uint32_t>(p.batch_pad);
    v.scan_done = c.take<uint32_t>(p.batch_pad);
    v.qnorm = c.take<float>(p.batch_pad);
    v.qshift = c.take<float>(p.batch_pad);
    v.keep = c.take<float>(p.batch_pad);
    v.keep_halves = p.halves ? c.take<float>(p.batch_pad) : nullptr;
    v.edge = c.take<float>(p.batch_pad);
    v.best_count = c.take<uint32_t>(p.batch_pad);
    v.qfrag = c.take<uint16_t>((size_t)p.batch_pad * p.KS * 16 * 2);
    v.qbytes = p.stationary ? c.take<uint8_t>((size_t)p.batch_pad * p.KS * 16) : nullptr;
    v.qhalf = p.halves ? c.take<uint16_t>((size_t)p.batch_pad * p.KS * 16) : nullptr;
    v.dense = c.take<float>((size_t)p.batch_pad * kDense);
    v.seg_count = c.take<uint32_t>((size_t)p.batch_pad * p.segs);
    v.lists = c.take<uint2>((size_t)p.batch * p.segs * p.seg_cap);
    v.best = c.take<unsigned long long>((size_t)p.batch * kBest);
    v.parts = c.take<unsigned long long>((size_t)p.scan_grid * p.scan_queries * k);
    if (a) *a = v;
    return c.used;
}

template <typename Elem, bool DENSE>
void launch_filter(const Plan& p, const BruteArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)(p.splits * p.groups)), block(kBfThreads);
    if (p.stationary && p.KS == 6) {
        hipLaunchKernelGGL((bf_filter_stationary_kernel<6, DENSE>), grid, block, 0, s, a);
    } else if (p.stationary) {
        hipLaunchKernelGGL((bf_filter_stationary_kernel<8, DENSE>), grid, block, 0, s, a);
    } else {
        hipLaunchKernelGGL((bf_filter_kernel<Elem, DENSE>), grid, block, 0, s, a);
        if (!DENSE && p.halves) hipLaunchKernelGGL(bf_halves_kernel, dim3((unsigned)(p.splits_halves * ((p.groups + 1) / 2))), dim3(2 * kBfThreads), 0, s, a);
    }
}

template <typename Elem>
hipError_t run(const Plan& p, BruteArgs a, const float* queries, int64_t nq, int64_t* out_ids, float* out_dists, hipStream_t s) {
    const size_t select_lds = sizeof(unsigned long long) * kDense + sizeof(float) * a.D;
    hipError_t e;
    if (select_lds + 8192 > 64 * 1024)
        if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(bf_select_kernel<Elem>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)select_lds)) != hipSuccess) return e;
    for (int64_t b0 = 0; b0 < nq; b0 += p.batch) {
        a.nq = nq - b0 < p.batch ? nq - b0 : p.batch;
        a.queries = queries + (size_t)b0 * a.D;
        a.out_ids = out_ids + (size_t)b0 * a.k;
        a.out_dists = out_dists + (size_t)b0 * a.k;
        // A crowded query may end in the exact scan, about 30 us in a large batch (1M x 128 floats) and 300 by itself, of which halves
        // save 0.4 a query: one in 128, none in a small batch, whose few queries are hardly ever taken for crowded by chance.
        a.crowded_most = a.nq < 1024 ? 0u : (uint32_t)(a.nq / 128);
        hipLaunchKernelGGL(pack_queries_kernel, dim3((unsigned)(p.batch_pad / 32)), dim3(a.KS < 16 ? 256 : 1024), 0, s, a);
        if (p.halves) {
            const int64_t count = p.batch_pad / 32 * p.KS * kWave;
            hipLaunchKernelGGL(pack_halves_kernel, dim3((unsigned)((count + kBfThreads - 1) / kBfThreads)), dim3(kBfThreads), 0, s, a, count);
        }
        for (uint64_t pos = 0; pos < a.N;) {
            const bool dense = pos == 0;
            uint64_t rows = dense ? (uint64_t)kDense : (uint64_t)((double)pos * (p.growth - 1.0));
            if (rows < (uint64_t)kDense) rows = kDense;
            if (rows > a.N - pos) rows = a.N - pos;
            a.chunk_pos = pos;
            a.chunk_rows = (int64_t)rows;
            // tiles of bytes: smaller where there would be fewer than workgroups
            a.tile_rows = kByteRows;
            while (a.tile_rows > 32 && rows < (uint64_t)a.tile_rows * p.splits) a.tile_rows /= 2;
            if (dense) launch_filter<Elem, true>(p, a, s);
            else launch_filter<Elem, false>(p, a, s);
            pos += rows;
            // Entries up to the end of the rank-th's bin that need no division of the bin, which takes a small batch a microsecond:
            // what they cost is an exact distance each, or, before the last chunk, the pairs that pass (see make_plan).
            const bool last = pos >= a.N;
            const int rank = rank_at(a.k, (double)pos, (double)a.N), least = rank + rank / 8 + 3;
            const int room = std::min(rank + 64, (int)(1600.0 / p.growth));
            const uint32_t few = (uint32_t)(last ? a.k + 128 : (a.nq < 1024 ? std::max(least, room) : least));
            hipLaunchKernelGGL((bf_select_kernel<Elem>), dim3((unsigned)a.nq), dim3(kBfThreads), select_lds, s, a, dense ? 1 : 0, last ? 1 : 0, rank, few);
        }
        const dim3 scan((unsigned)p.scan_grid), block(kBfThreads);
        if (p.scan_queries == 1) hipLaunchKernelGGL((bf_scan_kernel<Elem, 1>), scan, block, scan_lds(1, a.D), s, a);
        else hipLaunchKernelGGL((bf_scan_kernel<Elem, kScanQueries>), scan, block, scan_lds(kScanQueries, a.D), s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

size_t brute_force_workspace(int64_t nq, uint64_t N, int D, int elem_bytes, int k) {
    return carve(make_plan(nq, N, D, elem_bytes, k), k, nullptr, nullptr);
}

uint64_t brute_force_step(uint64_t N) {
    uint64_t step = (uint64_t)((double)N * 0.6180339887498949) | 1u;
    while (gcd_u64(step, N) != 1) step += 2;
    return step;
}

size_t brute_force_norm_words(uint64_t N, int D, int elem_bytes) { return elem_bytes == 1 ? centre_at(N) + (size_t)N : halves_at(N, D) + (size_t)N; }

hipError_t launch_half_norms(const void* vectors, int elem_bytes, uint64_t N, int D, float* out, hipStream_t s) {
    const dim3 grid((unsigned)(N / 16 + 1 < 2048 ? N / 16 + 1 : 2048)), block(kBfThreads);
    const pqt_host::BruteError err = pqt_host::brute_error(elem_bytes, D), half = pqt_host::brute_error_half(D);
    float* centre = out + centre_at(N);
    hipLaunchKernelGGL(clear_words_kernel, dim3(1), dim3(3), 0, s, reinterpret_cast<uint32_t*>(out) + N);
    if (elem_bytes == 1) {
        hipLaunchKernelGGL(half_norms_kernel<uint8_t>, grid, block, 0, s, static_cast<const uint8_t*>(vectors), (int64_t)N, D, centre, err, half, out, reinterpret_cast<int*>(centre), nullptr);
    } else {
        const float* x = static_cast<const float*>(vectors);
        const uint64_t step = brute_force_step(N);
        hipLaunchKernelGGL(centre_kernel, dim3((unsigned)((D + kWave - 1) / kWave)), block, 0, s, x, N, step, D, centre);
        hipLaunchKernelGGL(use_centre_kernel, dim3(1), dim3(1024), 0, s, x, N, step, D, centre, reinterpret_cast<uint32_t*>(out) + N + 1, out + N + 2);
        hipLaunchKernelGGL(half_norms_kernel<float>, grid, block, 0, s, x, (int64_t)N, D, centre, err, half, out, nullptr, out + halves_at(N, D));
    }
    return hipGetLastError();
}

hipError_t launch_brute_force(const void* vectors, const float* half_norms, int elem_bytes, uint64_t N, int D, const float* queries,
                              int64_t nq, int k, void* workspace, int64_t* out_ids, float* out_dists, hipStream_t s) {
    const Plan p = make_plan(nq, N, D, elem_bytes, k);
    BruteArgs a;
    carve(p, k, static_cast<unsigned char*>(workspace), &a);
    a.vectors = vectors; a.xhalf = half_norms; a.N = N; a.D = D; a.k = k; a.KS = p.KS;
    a.centre = elem_bytes == 4 ? half_norms + centre_at(N) : nullptr;
    a.ihalf = elem_bytes == 1 ? reinterpret_cast<const int*>(half_norms + centre_at(N)) : nullptr;
    a.use_centre = reinterpret_cast<const uint32_t*>(half_norms) + N + 1;
    a.splits = p.splits; a.splits_halves = p.splits_halves; a.segs = p.segs; a.seg_cap = p.seg_cap;
    a.crowded_next = (int)(kBest / p.growth);
    a.step = brute_force_step(N);
    a.err = pqt_host::brute_error(elem_bytes, D);
    a.err_half = pqt_host::brute_error_half(D);
    a.xhalf_halves = elem_bytes == 4 ? half_norms + halves_at(N, D) : nullptr;
    return elem_bytes == 1 ? run<uint8_t>(p, a, queries, nq, out_ids, out_dists, s) : run<float>(p, a, queries, nq, out_ids, out_dists, s);
}

}  // namespace pqt
