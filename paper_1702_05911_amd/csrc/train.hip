// Training on a sample (Sec. 3.1 "Training the codebook"; Sec. 3.3 "Offline computation"): the level-1
// product quantiser of every tree part by Lloyd iterations (Sec. 2.1), then, independently inside each
// of its cells, the level-2 quantiser of the sub-vectors that fall into the cell -- all k1 cells of a
// part are trained side by side as "groups" of one batched Lloyd run -- and the table of 256 line code
// points (i, j, lambda) per re-rank sub-part: every training sub-vector votes for the nearest line
// through two level-1 centroids (its projection error comes from its own level-1 distances, as in the
// re-ranking: b^2 - lambda^2 c^2 with lambda = (b^2 - a^2 + c^2) / (2 c^2)); lines receive code points
// in proportion to their votes, placed at the quantiles of the lambdas seen on the line.
//
// Everything per vector runs in the kernels below.  Results do not depend on the order in which the
// hardware schedules work: assignments break ties by the smaller centroid number, cell sums are taken
// over the members in ascending vector order in fixed chunks (double precision), re-seeding takes the
// farthest vector with the smallest number.

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "pqt_device.hpp"
#include "pqt_host.hpp"
#include "pqt_index.hpp"

using pqt_host::DeviceGuard;
using pqt_host::fail;

namespace pqt {
namespace {

constexpr int kTrainThreads = 256;
constexpr int kTile = kTrainThreads;       // vectors a workgroup works on at a time, one per thread
constexpr int kSlab = 32;                  // dimensions staged in LDS at a time
constexpr int kSlabStride = kSlab + 4;     // a lane's 16-byte reads fall into different banks
constexpr uint32_t kMaxChunks = 2048;      // chunks of vectors aimed at: eight workgroups per compute unit

__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), off, kWave);
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, off, kWave);
        const unsigned long long o = ((unsigned long long)hi << 32) | lo;
        v = o < v ? o : v;
    }
    return v;
}

// One batch of Lloyd runs: G groups of k centroids each, G / P groups per tree part.  Level 1 has one group per part (all
// vectors), level 2 one per level-1 cell.  Vectors are named by their position in their part's member list.
struct LloydArgs {
    const float* X;              // n x D
    uint64_t n;
    int D, dp, P, G, k;
    int kp;                      // k rounded up to the centroids a thread works on at a time
    int wide;                    // rows and slices are 16-byte aligned
    const uint32_t* members;     // [P][n]: position -> vector number (ascending inside a group); null: the same
    const uint2* range;          // [G]: the group's positions
    const uint32_t* chunk_off;   // [G + 1]: the group's chunks
    const uint4* chunks;         // (group, first position, end): consecutive pieces of a group
    uint8_t* frozen;             // [G]
    float* cen;                  // [G][k][dp]
    float* cenI;                 // [G][ceil(dp / 4)][kp][4]: four dimensions of all centroids side by side
    double* sums;                // [chunk][k][dp]
    uint32_t* counts;            // [chunk][k]
    float* dmin;                 // [P][n]
    uint32_t* label;             // [P][n]: written instead of sums when not null
};

__device__ __forceinline__ void put_centroid(const LloydArgs& g, int grp, int j, int d, float v) {
    g.cen[((size_t)grp * g.k + j) * g.dp + d] = v;
    g.cenI[(((size_t)grp * ((g.dp + 3) / 4) + d / 4) * g.kp + j) * 4 + d % 4] = v;
}

// Start centroids of every group (Sec. 2.1: Lloyd iterations need a start): k members at evenly spaced
// places of the group's member list.  A group with no more than k members is frozen: its members are
// centroids themselves, the remaining centroids repeat the members' mean (the parent centroid when
// the group is empty).  One workgroup per group.
__global__ __launch_bounds__(kTrainThreads) void lloyd_init_kernel(LloydArgs g, const float* parent) {
    const int grp = blockIdx.x, tid = threadIdx.x, dp = g.dp, k = g.k;
    const int p = grp / (g.G / g.P), col0 = p * dp;
    const uint2 rg = g.range[grp];
    const uint32_t ng = rg.y - rg.x;
    const uint32_t* mem = g.members ? g.members + (size_t)p * g.n : nullptr;
    if (tid == 0) g.frozen[grp] = ng <= (uint32_t)k ? 1 : 0;
    const size_t words = (size_t)((dp + 3) / 4) * g.kp * 4;       // the padding stays zero
    for (size_t e = tid; e < words; e += kTrainThreads) g.cenI[(size_t)grp * words + e] = 0.0f;
    __syncthreads();
    for (int e = tid; e < k * dp; e += kTrainThreads) {
        const int j = e / dp, d = e - j * dp;
        float v;
        if (ng > (uint32_t)k) {
            const uint32_t at = rg.x + (uint32_t)(((unsigned long long)j * ng) / (unsigned)k);
            v = g.X[(size_t)(mem ? mem[at] : at) * g.D + col0 + d];
        } else if ((uint32_t)j < ng) {
            v = g.X[(size_t)(mem ? mem[rg.x + j] : rg.x + j) * g.D + col0 + d];
        } else if (ng == 0) {
            v = parent ? parent[(size_t)grp * dp + d] : 0.0f;
        } else {
            double s = 0.0;
            for (uint32_t r = rg.x; r < rg.y; ++r) s += (double)g.X[(size_t)(mem ? mem[r] : r) * g.D + col0 + d];
            v = (float)(s / (double)ng);
        }
        put_centroid(g, grp, j, d, v);
    }
}

// The chunks of every group: pieces of `rows` members.  One workgroup; at most 1024 groups (four parts, 256 cells).
__global__ __launch_bounds__(1024) void chunk_table_kernel(const uint2* range, int G, uint32_t rows, uint32_t limit, uint32_t* chunk_off, uint4* chunks) {
    __shared__ uint32_t part[1024 / kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const uint2 mine = tid < G ? range[tid] : make_uint2(0u, 0u);
    uint32_t total;
    const uint32_t at = block_exclusive_sum((uint32_t)(((uint64_t)(mine.y - mine.x) + rows - 1) / rows), part, total);
    if (tid < G) chunk_off[tid] = at;
    if (tid == 0) chunk_off[G] = total;
    for (uint32_t c = total + tid; c < limit; c += blockDim.x) chunks[c] = make_uint4(0u, 0u, 0u, 0u);     // empty ones
    for (int l = 0; l < kWave; ++l) {                        // a wavefront writes its groups one after the other
        const int grp = wave * kWave + l;
        if (grp >= G) break;
        const uint32_t lo = (uint32_t)__shfl((int)mine.x, l, kWave), hi = (uint32_t)__shfl((int)mine.y, l, kWave);
        const uint32_t first = (uint32_t)__shfl((int)at, l, kWave);
        for (uint64_t c = lane, s = (uint64_t)lo + (uint64_t)lane * rows; s < hi; c += kWave, s += (uint64_t)kWave * rows)
            chunks[first + c] = make_uint4((uint32_t)grp, (uint32_t)s, (uint32_t)(s + rows < hi ? s + rows : hi), 0u);
    }
}

// One Lloyd iteration over one chunk: the nearest centroid of every vector among the k of its group (plain sums of squared
// differences, dimensions in ascending order; ties go to the smaller centroid number), then the sum and number of
// the members of every cell, in double precision, members in ascending order in a fixed split.
// A thread has one vector, whose values come from LDS 32 dimensions at a time, and KB running distances; the
// centroids are the same for the whole workgroup and come through the scalar cache.  The sums are taken from the vectors
// once more (they are in L2): the tile's vectors are ordered by cell, a wavefront adds up one cell's.  For rows and cells that
// lloyd_tile_kernel, below, has no room for, and where it is the slower one (tile_block).
// WAYS: 1, or 4 where there are too few vectors to fill the chip and many centroids (see ways_of): a tile is then 64
// vectors, and every wavefront has all of them and a quarter of the centroids.
template <int KB, int WAYS>
__global__ __launch_bounds__(kTrainThreads) void lloyd_step_kernel(LloydArgs g) {
    typedef const __attribute__((address_space(4))) float* scalar_floats;
    constexpr int TILE = kTile / WAYS;
    static_assert(WAYS == 1 || TILE == kWave, "a wavefront has one share of the centroids");
    __shared__ __align__(16) float sx[TILE * kSlabStride];
    __shared__ uint32_t srow[TILE], order[TILE], part[kTrainThreads / kWave];
    __shared__ unsigned long long nearest[WAYS > 1 ? TILE : 1];
    extern __shared__ uint32_t cnt[];                        // [wavefront][cell]: members, then their first place in `order`
    if (blockIdx.x >= g.chunk_off[g.G]) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    constexpr int nwaves = kTrainThreads / kWave;
    const uint4 chunk = g.chunks[blockIdx.x];
    const int grp = __builtin_amdgcn_readfirstlane((int)chunk.x);
    const uint32_t lo = chunk.y, hi = chunk.z;
    if (!g.label && g.frozen[grp]) return;
    const int dp = g.dp, k = g.k, nd4 = (dp + 3) / 4;
    const int p = grp / (g.G / g.P), col0 = p * dp;
    const uint32_t* mem = g.members ? g.members + (size_t)p * g.n : nullptr;
    const int way = WAYS > 1 ? wave : 0, mine = WAYS > 1 ? lane : tid;       // share of the centroids, vector of the tile
    for (uint64_t t0 = lo; t0 < hi; t0 += TILE) {
        const int m = (int)(hi - t0 < TILE ? hi - t0 : TILE);
        if (tid < m) srow[tid] = mem ? mem[t0 + tid] : (uint32_t)t0 + (uint32_t)tid;
        if (WAYS > 1 && tid < TILE) nearest[tid] = ~0ull;
        for (int e = tid; e < nwaves * k; e += kTrainThreads) cnt[e] = 0u;
        uint32_t best = 0xffffffffu, cell = 0u;
        bool first = true;
        for (int first_j = 0; first_j < k; first_j += KB * WAYS) {
            const int j0 = first_j + way * KB;               // (past the last: nothing to do but bring vectors)
            float acc[KB];
#pragma unroll
            for (int j = 0; j < KB; ++j) acc[j] = 0.0f;
            for (int d0 = 0; d0 < dp; d0 += kSlab) {
                __syncthreads();
                if (first || dp > kSlab) {
                    if (g.wide) {
                        // all pieces are asked for before the first is waited for: what a thread may not read it reads from the
                        // start of a row it may
                        float4 v[kSlab / 4 / WAYS];
#pragma unroll
                        for (int u = 0; u < kSlab / 4 / WAYS; ++u) {
                            const int e = tid + u * kTrainThreads, r = e / (kSlab / 4), d = d0 + 4 * (e % (kSlab / 4));
                            v[u] = *reinterpret_cast<const float4*>(g.X + (size_t)srow[r < m ? r : 0] * g.D + col0 + (d < dp ? d : 0));
                        }
#pragma unroll
                        for (int u = 0; u < kSlab / 4 / WAYS; ++u) {
                            const int e = tid + u * kTrainThreads, r = e / (kSlab / 4), d = d0 + 4 * (e % (kSlab / 4));
                            if (r >= m || d >= dp) v[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                            *reinterpret_cast<float4*>(sx + r * kSlabStride + (d - d0)) = v[u];
                        }
                    } else {
                        for (int e = tid; e < TILE * kSlab; e += kTrainThreads) {
                            const int r = e / kSlab, d = d0 + e % kSlab;
                            sx[r * kSlabStride + (d - d0)] = r < m && d < dp ? g.X[(size_t)srow[r] * g.D + col0 + d] : 0.0f;
                        }
                    }
                }
                first = false;
                __syncthreads();
                const int steps = WAYS == 1 || j0 < k ? min(kSlab / 4, nd4 - d0 / 4) : 0;
                scalar_floats c = (scalar_floats)(uintptr_t)(g.cenI + (((size_t)grp * nd4 + d0 / 4) * g.kp + j0) * 4);
                for (int s = 0; s < steps; ++s, c += (size_t)g.kp * 4) {
                    const float4 x = *reinterpret_cast<const float4*>(sx + mine * kSlabStride + 4 * s);
#pragma unroll
                    for (int j = 0; j < KB; ++j) {
                        float diff = x.x - c[4 * j];
                        acc[j] = fmaf(diff, diff, acc[j]);
                        diff = x.y - c[4 * j + 1];
                        acc[j] = fmaf(diff, diff, acc[j]);
                        diff = x.z - c[4 * j + 2];
                        acc[j] = fmaf(diff, diff, acc[j]);
                        diff = x.w - c[4 * j + 3];
                        acc[j] = fmaf(diff, diff, acc[j]);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                const uint32_t key = mono_key(acc[j]);
                if (j0 + j < k && (key < best || (j == 0 && first_j == 0))) {
                    best = key;
                    cell = (uint32_t)(j0 + j);
                }
            }
        }
        if (WAYS > 1) {                                      // the smallest (distance, centroid) of all shares
            if (way * KB < k) atomicMin(&nearest[mine], ((unsigned long long)best << 32) | cell);
            __syncthreads();
            best = (uint32_t)(nearest[mine] >> 32);
            cell = (uint32_t)nearest[mine];
        }
        if (tid < m) g.dmin[(size_t)p * g.n + t0 + tid] = mono_inv(best);
        if (g.label) {
            if (tid < m) g.label[(size_t)p * g.n + t0 + tid] = cell;
            if (WAYS > 1) __syncthreads();                   // (nearest[] has been read)
            continue;
        }
        // ---- the tile's vectors ordered by cell: a lane's place among the same cell's of its wavefront, then the counts ----
        unsigned long long same = __ballot(tid < m);
        for (int b = 1; b < k; b <<= 1) {
            const unsigned long long set = __ballot((cell & (uint32_t)b) != 0u);
            same &= (cell & (uint32_t)b) ? set : ~set;
        }
        const int before = __popcll(same & ((1ull << lane) - 1ull));
        if (tid < m && before == 0) cnt[wave * k + (int)cell] = (uint32_t)__popcll(same);
        __syncthreads();
        const int per = (k + kTrainThreads - 1) / kTrainThreads;
        uint32_t here = 0, total;
        for (int j = tid * per; j < min(k, (tid + 1) * per); ++j)
            for (int w = 0; w < nwaves; ++w) here += cnt[w * k + j];
        uint32_t place = block_exclusive_sum(here, part, total);
        for (int j = tid * per; j < min(k, (tid + 1) * per); ++j)
            for (int w = 0; w < nwaves; ++w) {
                const uint32_t c = cnt[w * k + j];
                cnt[w * k + j] = place;
                place += c;
            }
        __syncthreads();
        if (tid < m) order[cnt[wave * k + (int)cell] + (uint32_t)before] = srow[tid];
        __syncthreads();
        // ---- sums: one wavefront per cell and piece of the dimensions; several vectors side by side when the piece is short ----
        const bool more = t0 != lo;                          // a later tile adds to what the first one wrote
        const int units = g.wide ? dp / 4 : dp;
        int span = 1;
        while (span < units && span < kWave) span <<= 1;
        const int pieces = (units + span - 1) / span, rl = kWave / span, r = lane / span, dl = lane & (span - 1);
        for (int job = wave; job < k * pieces; job += nwaves) {
            const int j = job / pieces, unit = (job - j * pieces) * span + dl;
            const int a = (int)cnt[j], b = j + 1 < k ? (int)cnt[j + 1] : m;
            double* out = g.sums + ((size_t)blockIdx.x * k + j) * dp;
            if (g.wide) {
                const float* col = g.X + col0 + 4 * (unit < units ? unit : 0);
                double acc[4] = {0.0, 0.0, 0.0, 0.0};
                constexpr int kFlight = 8;                   // rows asked for before the first is waited for
                for (int e0 = a; e0 < b; e0 += kFlight * rl) {
                    float4 v[kFlight];
#pragma unroll
                    for (int u = 0; u < kFlight; ++u)
                        v[u] = *reinterpret_cast<const float4*>(col + (size_t)order[min(e0 + u * rl + r, b - 1)] * g.D);
#pragma unroll
                    for (int u = 0; u < kFlight; ++u)
                        if (e0 + u * rl + r < b) {
                            acc[0] += (double)v[u].x;
                            acc[1] += (double)v[u].y;
                            acc[2] += (double)v[u].z;
                            acc[3] += (double)v[u].w;
                        }
                }
                for (int off = span; off < kWave; off <<= 1)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] += __shfl_xor(acc[c], off, kWave);
                if (r == 0 && unit < units)
#pragma unroll
                    for (int c = 0; c < 4; ++c) out[4 * unit + c] = more ? out[4 * unit + c] + acc[c] : acc[c];
            } else {
                double acc = 0.0;
                if (unit < units)
                    for (int e = a + r; e < b; e += rl) acc += (double)g.X[(size_t)order[e] * g.D + col0 + unit];
                for (int off = span; off < kWave; off <<= 1) acc += __shfl_xor(acc, off, kWave);
                if (r == 0 && unit < units) out[unit] = more ? out[unit] + acc : acc;
            }
            if (lane == 0 && job == j * pieces) {
                uint32_t* n = g.counts + (size_t)blockIdx.x * k + j;
                *n = more ? *n + (uint32_t)(b - a) : (uint32_t)(b - a);
            }
        }
        __syncthreads();
    }
}

// ---- the same step with whole rows and the centroids in LDS ----------------------------------------------------------
// A lane works on VR vectors (lane mod 16, and 16 further) and on every fourth centroid, so that with VR = 2 six 16-byte reads
// feed 64 vector instructions (16 centroids).  A cell's sum is taken from the staged rows by the one wavefront that owns the
// cell, members in ascending order, and stays in its registers from tile to tile.  Rows come to LDS without passing through
// registers, an odd number of 16-byte pieces apart: a vector per lane (16 bytes) and a dimension per lane (4 bytes) read without
// conflicts.
// 100,000 vectors x 128, P = 2, an iteration's step, this kernel and lloyd_step_kernel: 16 centroids 28.7 and 35.8 us, 8 centroids
// in each of 16 cells 21.6 and 22.8.  Of the 28.7: two vector instructions per value and centroid 10.4, the way to the first
// vectors and their staging 6, sums 5; the four workgroups of a compute unit go through these steps nearly together.  With the
// centroids through the scalar cache and a quarter of them per wavefront the distances waited for them (31 to 40 us, also with the next
// rows on their way); sums added up in LDS, a cell's rows found one by one, took twice as long.
constexpr int kTileWaves = kTrainThreads / kWave;
constexpr int kTileDims = 128, kTileCells = 48;              // at most
constexpr int tile_vectors(int dp) { return dp <= kWave ? 2 : 1; }       // of a lane: the tile leaves room for three workgroups and more
struct TileLds {
    int st;                                                  // 16-byte pieces from row to row
    size_t cen, cell, row, list, total;
};
// kp: centroids of a group with the padding
__host__ __device__ constexpr TileLds tile_layout(int dp, int kp, int vr) {
    TileLds L = {};
    const int rows = kTileWaves * 16 * vr;
    L.st = (dp + 3) / 4 | 1;
    L.cen = (size_t)rows * L.st * 16;
    L.cell = L.cen + (size_t)((dp + 3) / 4) * kp * 16;
    L.row = L.cell + sizeof(uint32_t) * rows;
    L.list = L.row + sizeof(uint32_t) * rows;                // of every wavefront: rows by cell
    L.total = L.list + (size_t)kTileWaves * rows;
    return L;
}

// KR: centroids of a lane, and cells of a wavefront.  VR: vectors of a lane.  ND: dimensions of a lane when sums are taken.
template <int KR, int VR, int ND>
__global__ __launch_bounds__(kTrainThreads, 4) void lloyd_tile_kernel(LloydArgs g) {
    typedef const __attribute__((address_space(1))) void global_bytes;
    typedef __attribute__((address_space(3))) void lds_bytes;
    constexpr int kRows = kTileWaves * 16 * VR;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint4 chunk = g.chunks[blockIdx.x];
    const int grp = __builtin_amdgcn_readfirstlane((int)chunk.x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)chunk.y), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)chunk.z);
    if (lo == hi) return;                                    // past the last chunk
    if (!g.label && g.frozen[grp]) return;
    const int dp = g.dp, k = g.k, kp = g.kp, nd4 = (dp + 3) / 4;
    const int p = grp / (g.G / g.P), col0 = p * dp;
    const uint32_t* mem = g.members ? g.members + (size_t)p * g.n : nullptr;
    const TileLds L = tile_layout(dp, kp, VR);
    const int st = L.st;
    const float per_row = 1.0f / (float)st;
    float* sx = reinterpret_cast<float*>(smem);
    float4* cen = reinterpret_cast<float4*>(smem + L.cen);
    uint32_t* cells = reinterpret_cast<uint32_t*>(smem + L.cell);
    uint32_t* rows = reinterpret_cast<uint32_t*>(smem + L.row);
    uint8_t* list = smem + L.list + wave * kRows;
    // the vector of this thread's row of the tile at t0; what lies past the last one is read from there and not used
    // (64 bits: the last tile may end past 2^32)
    auto row_of = [&](uint64_t t0) {
        const uint32_t at = (uint32_t)min(t0 + (uint64_t)min(tid, kRows - 1), (uint64_t)hi - 1);
        return mem ? mem[at] : at;
    };
    uint32_t row = row_of(lo);
    const float4* from = reinterpret_cast<const float4*>(g.cenI) + (size_t)grp * nd4 * kp;
    for (int e = tid; e < nd4 * kp; e += kTrainThreads) cen[e] = from[e];
    double acc[KR][ND];
    uint32_t cnt[KR];
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        cnt[j] = 0u;
#pragma unroll
        for (int d = 0; d < ND; ++d) acc[j][d] = 0.0;
    }
    const int v0 = wave * 16 * VR + (lane & 15), column = lane >> 4;
    const float4* xs = reinterpret_cast<const float4*>(sx) + v0 * st;
    for (uint64_t t0 = lo; t0 < hi; t0 += kRows) {
        const int m = (int)min(hi - t0, (uint64_t)kRows);
        if (tid < kRows) rows[tid] = row;
        __syncthreads();                                     // (and the tile before is done with)
        row = row_of(t0 + kRows);
        // piece e of the tile is piece e mod st of row e / st
        if (g.wide) {
            for (int u = wave; u < kRows * st / kWave; u += kTileWaves) {
                const int e = u * kWave + lane, r = (int)(((float)e + 0.5f) * per_row), c = e - r * st;
                __builtin_amdgcn_global_load_lds((global_bytes*)(g.X + (size_t)rows[r] * g.D + col0 + 4 * (c < nd4 ? c : 0)),
                                                 (lds_bytes*)(sx + (size_t)u * kWave * 4), 16, 0, 0);
            }
        } else {
            for (int e = tid; e < kRows * nd4 * 4; e += kTrainThreads) {
                const int r = e / (nd4 * 4), d = e - r * (nd4 * 4);
                sx[r * st * 4 + d] = d < dp ? g.X[(size_t)rows[r] * g.D + col0 + d] : 0.0f;
            }
        }
        __builtin_amdgcn_s_waitcnt(0);                       // (the loads that write LDS)
        __syncthreads();
        if (wave * 16 * VR < m) {                            // the same for the wavefront
            float dist[VR][KR];
#pragma unroll
            for (int j = 0; j < KR; ++j)
#pragma unroll
                for (int v = 0; v < VR; ++v) dist[v][j] = 0.0f;
            const float4* c = cen + column;                  // this lane's centroids: column, column + 4, ...
#pragma unroll 2
            for (int s = 0; s < nd4; ++s) {
                float4 x[VR];
#pragma unroll
                for (int v = 0; v < VR; ++v) x[v] = xs[16 * v * st + s];
#pragma unroll
                for (int j = 0; j < KR; ++j) {
                    const float4 y = c[s * kp + 4 * j];
#pragma unroll
                    for (int v = 0; v < VR; ++v) {
                        float diff = x[v].x - y.x;
                        dist[v][j] = fmaf(diff, diff, dist[v][j]);
                        diff = x[v].y - y.y;
                        dist[v][j] = fmaf(diff, diff, dist[v][j]);
                        diff = x[v].z - y.z;
                        dist[v][j] = fmaf(diff, diff, dist[v][j]);
                        diff = x[v].w - y.w;
                        dist[v][j] = fmaf(diff, diff, dist[v][j]);
                    }
                }
            }
#pragma unroll
            for (int v = 0; v < VR; ++v) {
                unsigned long long best = ~0ull;
#pragma unroll
                for (int j = 0; j < KR; ++j) {
                    const unsigned long long key = ((unsigned long long)mono_key(dist[v][j]) << 32) | (uint32_t)(column + 4 * j);
                    if (column + 4 * j < k && key < best) best = key;
                }
                for (int off = 16; off < kWave; off <<= 1) {
                    const unsigned long long o = __shfl_xor(best, off, kWave);
                    best = o < best ? o : best;
                }
                const int r = v0 + 16 * v;
                if (column == 0) {
                    cells[r] = r < m ? (uint32_t)best : 0xffffffffu;
                    if (r < m) {
                        g.dmin[(size_t)p * g.n + t0 + r] = mono_inv((uint32_t)(best >> 32));
                        if (g.label) g.label[(size_t)p * g.n + t0 + r] = (uint32_t)best;
                    }
                }
            }
        } else if (lane < 16 * VR) {
            cells[wave * 16 * VR + lane] = 0xffffffffu;
        }
        __syncthreads();
        if (g.label) continue;
        // the rows of this wavefront's cells, in order, then their sums: four rows on their way
        constexpr int kHalves = kRows / kWave;
        uint32_t cell[kHalves];
        int first[KR + 1];
        first[0] = 0;
#pragma unroll
        for (int h = 0; h < kHalves; ++h) cell[h] = cells[h * kWave + lane];
#pragma unroll
        for (int j = 0; j < KR; ++j) {
            int n = first[j];
#pragma unroll
            for (int h = 0; h < kHalves; ++h) {
                const bool mine = cell[h] == (uint32_t)(wave + kTileWaves * j);
                const unsigned long long all = __ballot(mine);
                if (mine) list[n + __popcll(all & ((1ull << lane) - 1ull))] = (uint8_t)(h * kWave + lane);
                n += __popcll(all);
            }
            first[j + 1] = n;
            cnt[j] += (uint32_t)(n - first[j]);
        }
        wave_lds_order();
#pragma unroll
        for (int h = 0; h < kHalves; ++h) {                  // 64 places of the list at a time
            if (h * kWave >= first[KR]) break;
            const int place = (int)list[min(h * kWave + lane, first[KR] - 1)] * st * 4;
#pragma unroll
            for (int j = 0; j < KR; ++j) {
                const int from_i = max(first[j] - h * kWave, 0), to_i = min(first[j + 1] - h * kWave, kWave);
                for (int i = from_i; i < to_i; i += 4) {
                    float v[4][ND];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const float* x = sx + lane + __builtin_amdgcn_readlane(place, min(i + u, to_i - 1));
#pragma unroll
                        for (int d = 0; d < ND; ++d) v[u][d] = x[d * kWave];     // (past the row's end: not written out)
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (i + u < to_i)
#pragma unroll
                            for (int d = 0; d < ND; ++d) acc[j][d] += (double)v[u][d];
                }
            }
        }
    }
    if (g.label) return;
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        const int cell = wave + kTileWaves * j;
        if (cell >= k) continue;
        double* out = g.sums + ((size_t)blockIdx.x * k + cell) * dp;
#pragma unroll
        for (int d = 0; d < ND; ++d)
            if (lane + d * kWave < dp) out[lane + d * kWave] = acc[j][d];
        if (lane == 0) g.counts[(size_t)blockIdx.x * k + cell] = cnt[j];
    }
}

// Sum over the workgroup, returned to every thread.
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* part) {
    uint32_t total;
    (void)block_exclusive_sum(v, part, total);
    __syncthreads();
    return total;
}

// centroid = mean of its members (the chunks added in a fixed split and order); the cells of a frozen or empty
// group keep what they hold.  An empty cell is re-seeded with the member of its group that lies farthest from its
// centroid (ties: the smaller vector number); that vector then counts as at distance zero, so the next empty cell of the
// group takes another one.  One workgroup per cell and DIMS dimensions: 64, or 16 where that would be fewer workgroups than compute units
// (update_dims).
constexpr int kSeedDims = 64;
template <int DIMS>
__global__ __launch_bounds__(1024) void lloyd_update_kernel(LloydArgs g) {
    __shared__ double red[1024 / kWave * DIMS];
    __shared__ uint32_t part[1024 / kWave];
    __shared__ unsigned long long far_part[1024 / kWave];
    const int nt = blockDim.x, tid = threadIdx.x, lane = tid & (kWave - 1), k = g.k, dp = g.dp;
    const int grp = blockIdx.x / k, j = blockIdx.x - grp * k, p = grp / (g.G / g.P);
    const uint32_t c0 = g.chunk_off[grp], c1 = g.chunk_off[grp + 1];
    const uint8_t keep = g.frozen[grp];
    if (keep || c0 == c1) return;
    const int dl = lane & (DIMS - 1), d = blockIdx.y * DIMS + dl, r = tid / DIMS, rl = nt / DIMS;
    uint32_t mine = 0;
    for (uint32_t c = c0 + tid; c < c1; c += nt) mine += g.counts[(size_t)c * k + j];
    double acc = 0.0;
    constexpr int kFlight = 8;                               // chunks asked for before the first is waited for
    const double* col = g.sums + (size_t)j * dp + (d < dp ? d : 0);
    for (uint32_t e = c0; e < c1; e += kFlight * rl) {
        double v[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) v[u] = col[(size_t)min(e + u * rl + r, c1 - 1) * k * dp];
#pragma unroll
        for (int u = 0; u < kFlight; ++u)
            if (e + u * rl + r < c1) acc += v[u];
    }
    for (int off = DIMS; off < kWave; off <<= 1) acc += __shfl_xor(acc, off, kWave);
    if (lane < DIMS) red[tid / kWave * DIMS + lane] = acc;
    const uint32_t count = block_sum(mine, part);
    if (count > 0) {
        if (r == 0 && d < dp) {
            double t = 0.0;
            for (int s = 0; s < nt / kWave; ++s) t += red[s * DIMS + dl];
            put_centroid(g, grp, j, d, (float)(t / (double)count));
        }
        return;
    }
    // this is empty cell number `nth` of its group: it gets the nth farthest member, which one workgroup per kSeedDims dimensions looks for
    // (all of them: 100,000 vectors x 128, nineteen twentieths of them zero, 256 centroids 12.2 -> 20.4 ms), not the same of every cell and
    // piece, as every 256th workgroup is on the same compute unit
    constexpr int kSeeders = kSeedDims / DIMS;
    const int piece = blockIdx.y / kSeeders, seeders = min(kSeeders, (int)gridDim.y - piece * kSeeders);
    if ((int)blockIdx.y - piece * kSeeders != (j + piece) % seeders) return;
    const uint2 rg = g.range[grp];
    const float* dist = g.dmin + (size_t)p * g.n;
    int nth = 0;
    for (int i = 0; i < j; ++i) {
        uint32_t c_i = 0;
        for (uint32_t c = c0 + tid; c < c1; c += nt) c_i += g.counts[(size_t)c * k + i];
        if (block_sum(c_i, part) == 0) ++nth;
    }
    unsigned long long bound = ~0ull;
    uint32_t at = rg.x;                                      // none but zeros left: the first member
    for (int pass = 0; pass <= nth; ++pass) {
        unsigned long long best = 0ull;
        for (uint64_t e = (uint64_t)rg.x + tid; e < rg.y; e += nt) {
            const uint32_t dk = mono_key(dist[e]);
            const unsigned long long key = ((unsigned long long)dk << 32) | (0xffffffffu - (uint32_t)e);
            if (dk > mono_key(0.0f) && key < bound) best = key > best ? key : best;
        }
        best = ~wave_min_u64(~best);
        __syncthreads();
        if (lane == 0) far_part[tid / kWave] = best;
        __syncthreads();
        for (int s = 0; s < nt / kWave; ++s) best = far_part[s] > best ? far_part[s] : best;
        if (best == 0ull) {
            at = rg.x;
            break;
        }
        at = 0xffffffffu - (uint32_t)best;
        bound = best;
    }
    const float* x = g.X + (size_t)(g.members ? g.members[(size_t)p * g.n + at] : at) * g.D + (size_t)p * dp;
    const int e = piece * kSeedDims + tid;
    if (tid < kSeedDims && e < dp) put_centroid(g, grp, j, e, x[e]);
}

// ---- members of every part's cells, in ascending vector order ---------------------------------------------------------
// A count per piece of `rows` labels and cell, a prefix sum over (cell, piece), and every vector goes to its place: three short
// kernels (100,000 vectors, two parts: 14 us; a library sort of (label, vector) pairs per part took 100).
constexpr int kCellThreads = 1024;
constexpr int kCellWaves = kCellThreads / kWave;

// counts[p][cell][piece]; blockIdx.y = p
__global__ __launch_bounds__(kCellThreads) void cell_counts_kernel(const uint32_t* label, uint64_t n, int k, uint32_t rows, uint32_t* counts) {
    extern __shared__ uint32_t cnt[];
    const uint32_t* l = label + (size_t)blockIdx.y * n;
    for (int j = threadIdx.x; j < k; j += kCellThreads) cnt[j] = 0u;
    __syncthreads();
    const uint64_t r0 = (uint64_t)blockIdx.x * rows, r1 = min(n, r0 + rows);
    for (uint64_t r = r0 + threadIdx.x; r < r1; r += kCellThreads) atomicAdd(&cnt[l[r]], 1u);
    __syncthreads();
    for (int j = threadIdx.x; j < k; j += kCellThreads) counts[((size_t)blockIdx.y * k + j) * gridDim.x + blockIdx.x] = cnt[j];
}

// counts -> first places, in place; range[p * k + cell] = the cell's positions.  One workgroup per part.
__global__ __launch_bounds__(kCellThreads) void cell_places_kernel(uint32_t* counts, uint32_t n, int k, uint32_t pieces, uint2* range) {
    __shared__ uint32_t part[kCellWaves];
    const uint32_t items = (uint32_t)k * pieces;
    uint32_t* c = counts + (size_t)blockIdx.x * items;
    uint2* rg = range + (size_t)blockIdx.x * k;
    uint32_t before = 0;
    for (uint32_t e0 = 0; e0 < items; e0 += kCellThreads) {
        const uint32_t e = e0 + threadIdx.x;
        uint32_t total;
        const uint32_t at = before + block_exclusive_sum(e < items ? c[e] : 0u, part, total);
        before += total;
        if (e < items) {
            c[e] = at;
            if (e % pieces == 0) {
                rg[e / pieces].x = at;
                if (e > 0) rg[e / pieces - 1].y = at;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) rg[k - 1].y = n;
}

__global__ __launch_bounds__(kCellThreads) void cell_members_kernel(const uint32_t* label, uint64_t n, int k, uint32_t rows, const uint32_t* places,
                                                                    uint32_t* members) {
    extern __shared__ uint32_t lds[];
    uint32_t* next = lds;                                    // [cell]: its next place
    uint32_t* cnt = lds + k;                                 // [wavefront][cell]
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const uint32_t* l = label + (size_t)blockIdx.y * n;
    uint32_t* out = members + (size_t)blockIdx.y * n;
    for (int j = tid; j < k; j += kCellThreads) next[j] = places[((size_t)blockIdx.y * k + j) * gridDim.x + blockIdx.x];
    const uint64_t r0 = (uint64_t)blockIdx.x * rows, r1 = min(n, r0 + rows);
    for (uint64_t t0 = r0; t0 < r1; t0 += kCellThreads) {
        for (int j = tid; j < kCellWaves * k; j += kCellThreads) cnt[j] = 0u;
        __syncthreads();
        const bool have = t0 + tid < r1;
        const uint32_t cell = have ? l[t0 + tid] : 0u;
        unsigned long long same = __ballot(have);            // lanes with this lane's cell
        for (int b = 1; b < k; b <<= 1) {
            const unsigned long long set = __ballot((cell & (uint32_t)b) != 0u);
            same &= (cell & (uint32_t)b) ? set : ~set;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        if (have && rank == 0) cnt[wave * k + (int)cell] = (uint32_t)__popcll(same);
        __syncthreads();
        for (int j = tid; j < k; j += kCellThreads) {        // counts -> places of the wavefronts, in order
            uint32_t at = next[j];
            for (int w = 0; w < kCellWaves; ++w) {
                const uint32_t c = cnt[w * k + j];
                cnt[w * k + j] = at;
                at += c;
            }
            next[j] = at;
        }
        __syncthreads();
        if (have) out[cnt[wave * k + (int)cell] + (uint32_t)rank] = (uint32_t)(t0 + tid);
        __syncthreads();
    }
}

__global__ void whole_range_kernel(uint32_t n, int P, uint2* range) {
    if ((int)threadIdx.x < P) range[threadIdx.x] = make_uint2(0u, n);
}

// ---- the lambdas of every line's votes, and those at given ranks -----------------------------------------------------
// Only a few ranks of a line are wanted, so its votes are brought together but not sorted: counts per line, a place for every vote, and a radix
// select for the code points of a line (100,000 vectors x 8 sub-parts, 120 lines: 7, 10 and 22 us; a library sort of all votes took 160).  A
// workgroup of the first two takes kCellThreads votes of one sub-part; up to kLdsLines lines it counts in LDS and adds up or reserves once per
// line.
constexpr int kLdsLines = 8192;

__device__ __forceinline__ int vote_line(unsigned long long key) { return (int)((key >> 32) & 0xffffu); }

// One more in cnt[at] for every lane of the wavefront that has one; the count before it.  Where many lanes have the same, which additions to one
// address would take one after the other, the first lane's are added at once.
__device__ __forceinline__ uint32_t count_one(uint32_t* cnt, uint32_t at, bool have) {
    const int lane = threadIdx.x & (kWave - 1);
    const unsigned long long all = __ballot(have);
    if (all == 0ull) return 0u;
    const int first = __ffsll((long long)all) - 1;
    const bool mine = have && at == (uint32_t)__builtin_amdgcn_readlane((int)at, first);
    const unsigned long long same = __ballot(mine);
    uint32_t before = 0u;
    if (have && (!mine || lane == first)) before = atomicAdd(&cnt[at], mine ? (uint32_t)__popcll(same) : 1u);
    const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)before, first);
    return mine ? base + (uint32_t)__popcll(same & ((1ull << lane) - 1ull)) : before;
}

// The same without the count before it
__device__ __forceinline__ void add_one(uint32_t* cnt, uint32_t at, bool have) {
    const unsigned long long all = __ballot(have);
    if (all == 0ull) return;
    const int first = __ffsll((long long)all) - 1;
    const bool mine = have && at == (uint32_t)__builtin_amdgcn_readlane((int)at, first);
    const unsigned long long same = __ballot(mine);
    if (have && (!mine || (int)(threadIdx.x & (kWave - 1)) == first)) atomicAdd(&cnt[at], mine ? (uint32_t)__popcll(same) : 1u);
}

// count_one where all workgroups count in the same memory: what thread 0 has is added once for the workgroup (100,000 votes, nine tenths of them
// for one of 9,730 lines: vote_counts_kernel 117 -> 20 us, vote_groups_kernel 118 -> 21; spread over the lines 14 and 17).
__device__ __forceinline__ uint32_t count_one_of_block(uint32_t* cnt, uint32_t at, bool have) {
    __shared__ uint32_t before[kCellWaves], lead, base;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    if (tid == 0) lead = have ? at : 0xffffffffu;
    __syncthreads();
    const bool mine = have && at == lead;
    const unsigned long long same = __ballot(mine);
    if (lane == 0) before[wave] = (uint32_t)__popcll(same);
    __syncthreads();
    if (tid == 0) {
        uint32_t total = 0u;
        for (int w = 0; w < kCellWaves; ++w) {
            const uint32_t c = before[w];
            before[w] = total;
            total += c;
        }
        base = total ? atomicAdd(&cnt[lead], total) : 0u;
    }
    const uint32_t other = count_one(cnt, at, have && !mine);
    __syncthreads();
    return mine ? base + before[wave] + (uint32_t)__popcll(same & ((1ull << lane) - 1ull)) : other;
}

// counts[m][line]; votes without a line (number 0xffff) are not counted
__global__ __launch_bounds__(kCellThreads) void vote_counts_kernel(const unsigned long long* keys, uint32_t nt, int lines, uint32_t* counts) {
    extern __shared__ uint32_t cnt[];
    const int m = blockIdx.y, tid = threadIdx.x;
    const uint32_t v = blockIdx.x * kCellThreads + tid;
    const int line = v < nt ? vote_line(keys[(size_t)m * nt + v]) : 0xffff;
    uint32_t* out = counts + (size_t)m * lines;
    if (lines > kLdsLines) {
        (void)count_one_of_block(out, (uint32_t)line, line < lines);
        return;
    }
    for (int j = tid; j < lines; j += kCellThreads) cnt[j] = 0u;
    __syncthreads();
    add_one(cnt, (uint32_t)line, line < lines);
    __syncthreads();
    for (int j = tid; j < lines; j += kCellThreads)
        if (cnt[j]) atomicAdd(&out[j], cnt[j]);
}

// lam[m][next[m][line] ...]: the ordered bits of the line's lambdas, in any order; next: the line's first place at the start
__global__ __launch_bounds__(kCellThreads) void vote_groups_kernel(const unsigned long long* keys, uint32_t nt, int lines, uint32_t* next, uint32_t* lam) {
    extern __shared__ uint32_t cnt[];
    const int m = blockIdx.y, tid = threadIdx.x;
    const uint32_t v = blockIdx.x * kCellThreads + tid;
    const unsigned long long key = v < nt ? keys[(size_t)m * nt + v] : ~0ull;
    const int line = vote_line(key);
    uint32_t* places = next + (size_t)m * lines;
    uint32_t at = 0u;
    if (lines > kLdsLines) {
        at = count_one_of_block(places, (uint32_t)line, line < lines);
    } else {
        for (int j = tid; j < lines; j += kCellThreads) cnt[j] = 0u;
        __syncthreads();
        const uint32_t mine = count_one(cnt, (uint32_t)line, line < lines);
        __syncthreads();
        for (int j = tid; j < lines; j += kCellThreads)
            if (cnt[j]) cnt[j] = atomicAdd(&places[j], cnt[j]);
        __syncthreads();
        if (line < lines) at = cnt[line] + mine;
    }
    if (line < lines) lam[(size_t)m * nt + at] = (uint32_t)key;
}

// A job: code points of one line, at most kPicks of them; job = (first lambda of the line in its sub-part, lambdas, first code point of the job,
// code points), and sub-part m has the code points 256 m to 256 m + 255; lam holds the sub-parts from m0 on.  ranks[e]: the rank (from 0) of code
// point e among its line's lambdas, ascending within a job.  Eight bits a pass, the highest first.  The code points of a job that have the same
// bits so far are a group and share a histogram, so a pass reads the lambdas once whatever their number: a line with most of the votes has most of
// the 256 code points as well (pqt_train of 100,000 vectors, one iteration, with 16 centroids and nine tenths of the vectors zero 0.92 ms, a walk
// per code point 3.25; with one line 0.48 and 0.80, 2,000,000 vectors 1.25 and 9.5).
constexpr int kPicks = 32;
struct PickLds {
    uint32_t prefix[kPicks], start[kPicks + 1], rank[kPicks], digit[kPicks];      // of a group: its bits, its first code point
    uint32_t groups;
};

// By the first wavefront: the groups, from the bits that code point `lane` has so far.  Ranks ascend, so equal ones lie side by side.
__device__ __forceinline__ void group_picks(PickLds& s, uint32_t bits, int picks) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t left = (uint32_t)__shfl_up((int)bits, 1, kWave);
    const bool opens = lane < picks && (lane == 0 || bits != left);
    const unsigned long long all = __ballot(opens);
    const int groups = __popcll(all), mine = __popcll(all & ((1ull << lane) - 1ull));
    if (opens) {
        s.prefix[mine] = bits;
        s.start[mine] = (uint32_t)lane;
    }
    if (lane == 0) {
        s.start[groups] = (uint32_t)picks;
        s.groups = (uint32_t)groups;
    }
}

// By the workgroup: hist[group * 256 + digit] of the lambdas lo .. hi - 1.
__device__ __forceinline__ void count_digits(const PickLds& s, const uint32_t* x, uint64_t lo, uint64_t hi, int shift, uint32_t* hist) {
    const int tid = threadIdx.x, threads = blockDim.x, ng = (int)s.groups;
    int half = 1;
    while (2 * half < ng) half *= 2;
    constexpr int kFlight = 4;                               // lambdas asked for before the first is waited for
    for (uint64_t e0 = lo; e0 < hi; e0 += (uint64_t)kFlight * threads) {
        uint32_t key[kFlight];
        int g[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            key[u] = x[min(e0 + (uint64_t)(u * threads + tid), hi - 1)];
            g[u] = 0;
        }
        if (shift < 24) {                                    // the group with these bits, if there is one
            for (int step = half; step > 0; step /= 2)
#pragma unroll
                for (int u = 0; u < kFlight; ++u)
                    if (g[u] + step < ng && s.prefix[g[u] + step] <= key[u] >> (shift + 8)) g[u] += step;
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const bool have = e0 + (uint64_t)(u * threads + tid) < hi && (shift == 24 || s.prefix[g[u]] == key[u] >> (shift + 8));
            add_one(hist, (uint32_t)g[u] * 256u + ((key[u] >> shift) & 0xffu), have);
        }
    }
}

// By the workgroup: the next digit of every code point, and its rank among the lambdas that have it.  A wavefront per group, four counts a lane.
__device__ __forceinline__ void next_digits(PickLds& s, const uint32_t* hist) {
    const int lane = threadIdx.x & (kWave - 1);
    for (int g = (int)threadIdx.x / kWave; g < (int)s.groups; g += (int)blockDim.x / kWave) {
        const uint4 c = *reinterpret_cast<const uint4*>(hist + g * 256 + 4 * lane);
        uint32_t upto = c.x + c.y + c.z + c.w;
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)upto, off, kWave);
            if (lane >= off) upto += o;
        }
        const uint32_t a0 = upto - c.w - c.z - c.y, a1 = upto - c.w - c.z, a2 = upto - c.w;
        for (uint32_t t = s.start[g]; t < s.start[g + 1]; ++t) {
            const uint32_t rank = s.rank[t];
            if (lane == __popcll(__ballot(upto <= rank))) {
                const int d = (a0 <= rank) + (a1 <= rank) + (a2 <= rank);
                s.digit[t] = (uint32_t)(4 * lane + d);
                s.rank[t] = rank - (d == 0 ? a0 - c.x : (d == 1 ? a0 : (d == 2 ? a1 : a2)));
            }
        }
    }
}

// out[e]: the lambda of code point e, of a workgroup's job
constexpr int kPickThreads = 512;                            // (256: 29 us, 1,024: 28)
__global__ __launch_bounds__(kPickThreads) void pick_lambdas_kernel(const uint32_t* lam, uint32_t nt, uint32_t m0, const uint4* jobs,
                                                                    const uint32_t* ranks, float* out) {
    __shared__ __align__(16) uint32_t hist[kPicks * 256];
    __shared__ PickLds s;
    const int tid = threadIdx.x;
    const uint4 job = jobs[blockIdx.x];
    const uint32_t* x = lam + (size_t)(job.z / 256 - m0) * nt + job.x;
    const int picks = (int)job.w;
    uint32_t bits = 0u;                                      // of code point `tid`
    if (tid < picks) s.rank[tid] = ranks[job.z + tid];
    if (tid < kWave) group_picks(s, 0u, picks);
    __syncthreads();
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int e = tid; e < (int)s.groups * 256; e += blockDim.x) hist[e] = 0u;
        __syncthreads();
        count_digits(s, x, 0, job.y, shift, hist);
        __syncthreads();
        next_digits(s, hist);
        __syncthreads();
        if (tid < picks) bits = (bits << 8) | s.digit[tid];
        if (tid < kWave) group_picks(s, bits, picks);
        __syncthreads();
    }
    if (tid < picks) out[job.z + tid] = mono_inv(bits);
}

// The same for long lines, whose lambdas many workgroups read: a pass is two kernels (one line of 2,000,000 votes: 256 us instead of 3,800).  bits,
// ranks: of the code points, from pass to pass; counts[code point * 256 + digit]: the histograms of a job's groups are at its first code points,
// zero between passes. items: (job, slice)
__global__ __launch_bounds__(1024) void slice_digits_kernel(const uint32_t* lam, uint32_t nt, uint32_t m0, const uint4* jobs, const uint2* items,
                                                            uint32_t slice, int shift, const uint32_t* bits, uint32_t* counts) {
    __shared__ __align__(16) uint32_t hist[kPicks * 256];
    __shared__ PickLds s;
    const int tid = threadIdx.x;
    const uint2 item = items[blockIdx.x];
    const uint4 job = jobs[item.x];
    const int picks = (int)job.w;
    if (tid < kWave) group_picks(s, shift < 24 && tid < picks ? bits[job.z + tid] : 0u, picks);
    __syncthreads();
    const int cells = (int)s.groups * 256;
    for (int e = tid; e < cells; e += blockDim.x) hist[e] = 0u;
    __syncthreads();
    const uint64_t lo = (uint64_t)item.y * slice;
    count_digits(s, lam + (size_t)(job.z / 256 - m0) * nt + job.x, lo, min(lo + slice, (uint64_t)job.y), shift, hist);
    __syncthreads();
    for (int e = tid; e < cells; e += blockDim.x)
        if (hist[e]) atomicAdd(&counts[(size_t)job.z * 256 + e], hist[e]);
}

__global__ __launch_bounds__(256) void next_digits_kernel(const uint4* jobs, int shift, uint32_t* ranks, uint32_t* bits, uint32_t* counts,
                                                          float* out) {
    __shared__ PickLds s;
    const int tid = threadIdx.x;
    const uint4 job = jobs[blockIdx.x];
    const int picks = (int)job.w;
    uint32_t mine = shift < 24 && tid < picks ? bits[job.z + tid] : 0u;
    if (tid < picks) s.rank[tid] = ranks[job.z + tid];
    if (tid < kWave) group_picks(s, mine, picks);
    __syncthreads();
    uint32_t* c = counts + (size_t)job.z * 256;
    next_digits(s, c);
    __syncthreads();
    for (int e = tid; e < (int)s.groups * 256; e += 256) c[e] = 0u;
    if (tid >= picks) return;
    mine = (mine << 8) | s.digit[tid];
    bits[job.z + tid] = mine;
    ranks[job.z + tid] = s.rank[tid];
    if (shift == 0) out[job.z + tid] = mono_inv(mine);
}

__global__ void clear_counts_kernel(uint32_t* out, size_t n) {
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) out[e] = 0u;
}

// Everything pqt_train holds on the GPU: asked for first, then one allocation.
struct Arena {
    std::vector<std::pair<void**, size_t>> parts;
    size_t bytes = 0;
    void* base = nullptr;
    ~Arena() { (void)hipFree(base); }
    template <typename Tp>
    void want(Tp** out, size_t count) {
        parts.emplace_back(reinterpret_cast<void**>(out), bytes);
        bytes += (count * sizeof(Tp) + 255) / 256 * 256;
    }
    hipError_t allocate() {
        const hipError_t e = hipMalloc(&base, bytes ? bytes : 1);
        if (e == hipSuccess)
            for (const auto& p : parts) *p.first = static_cast<unsigned char*>(base) + p.second;
        return e;
    }
};

// Centroids a thread of lloyd_step_kernel works on at a time: a multiple of eight, at most 32 (its running distances are
// registers), so that the rounds over k leave less than eight of them unused each.
int centroid_block(int k) {
    const int rounds = (k + 31) / 32;
    return ((k + rounds - 1) / rounds + 7) / 8 * 8;
}

// Centroids of a lane of lloyd_tile_kernel; 0 where lloyd_step_kernel is the one to take: rows or cells beyond its registers and what leaves room
// for one workgroup per compute unit only, and where it is the faster one.  pqt_train, 10 iterations, level 1 only where one number of centroids is
// named, this kernel's time over the other's: Rows of few values with few centroids, whose distances are less than a tile's fixed steps: 1,000,000
// vectors x 4 with 1, 4, 8, 12 and 16 centroids 1.54, 1.29, 1.16, 1.05, 0.95; x 16 1.39, 1.20, 1.13, 1.03, 0.98; x 32 1.16, 1.07, 1.03, 0.94, 0.96;
// x 48 0.86 and less; 100,000 x 4 1.24, 1.15, 1.07, 1.00, 0.97, x 32 1.00, 1.11, 1.10, 0.88, 0.85; 60,000 x 8 1.07, 1.06, 1.04, 0.94, 0.94; 30,000
// x 8 0.94, 0.99, 1.00, 0.85, 0.84.  Not read in 16-byte pieces: 1,000,000 x 1 1.26, 1.08, 0.98, x 2 1.17, 0.91, 0.88. Long rows and many
// centroids, of which two workgroups share a compute unit, in so many groups that their last chunks are short: 128 dimensions, 40 centroids in each
// of 256 groups, 75,000 vectors 1.05, 100,000 1.09, 300,000 1.03; of 128 groups 0.91 to 1.03; 120 dimensions and less 0.87 to 1.00.
int tile_block(uint64_t n, int P, int G, int k, int dp) {
    if (dp > kTileDims || k > kTileCells) return 0;
    const uint64_t rows = (uint64_t)P * n;
    if (dp % 4 ? dp * k <= 4 && rows > (1u << 18) : (dp <= 16 ? k <= 12 && rows > (1u << 16) : dp <= 32 && k <= 8 && rows > 90'000)) return 0;
    if (dp > 120 && k > 32 && G > 128 && rows > (1u << 17)) return 0;
    const int want = (k + 3) / 4;
    const int kr = want <= 8 ? want : 12;
    return tile_layout(dp, 4 * kr, tile_vectors(dp)).total <= 64 * 1024 ? kr : 0;
}
int padded_centroids(uint64_t n, int P, int G, int k, int dp) {
    if (const int kr = tile_block(n, P, G, k, dp)) return 4 * kr;
    const int kb = centroid_block(k);
    return (k + kb - 1) / kb * kb;
}

// Shares of the centroids in lloyd_step_kernel: four where tiles of 256 vectors are fewer than the compute units and every
// wavefront gets a round of 32 centroids.  pqt_train of 128 dimensions, 256 centroids, 20 iterations, no line table: 20,000
// vectors 19.7 -> 14.2 ms, 5,000 vectors 19.7 -> 9.3 (one wavefront per vector: 14.7 and 10.0).
int ways_of(uint64_t n, int P, int k) { return k >= 128 && (uint64_t)P * ((n + kTile - 1) / kTile) < 256 ? 4 : 1; }

// Vectors per chunk (a workgroup of lloyd_step_kernel): one tile, or more where that would be more chunks than keep the
// chip busy, or more than 64 MB of cell sums.
uint64_t chunk_rows(uint64_t n, int P, int G, int k, int dp) {
    if (const int kr = tile_block(n, P, G, k, dp)) {
        // as many as the compute units hold at once (the last one of every group is a short one): at most 1,024, and some 50 MB of sums
        const uint64_t fit = std::min<uint64_t>(4, kMaxLds / tile_layout(dp, 4 * kr, tile_vectors(dp)).total);
        uint64_t want = 256 * fit;
        want -= std::min<uint64_t>((uint64_t)G, want / 2);
        const uint64_t rows = ((uint64_t)P * n + want - 1) / want;
        // (at least half a tile of 128; half and whole, 64 dimensions, 16 centroids: 10,000 vectors 396 and 436 us, 32,000 477 and 510, 50,000
        // 516 and 502)
        return std::max<uint64_t>(rows, 64);
    }
    uint64_t rows = kTile / ways_of(n, P, k);
    while (rows < n && rows < (1ull << 30) && ((uint64_t)P * ((n + rows - 1) / rows) > kMaxChunks ||
                        ((uint64_t)P * ((n + rows - 1) / rows) + (uint64_t)G) * (uint64_t)k * (uint64_t)dp > (8ull << 20)))
        rows *= 2;
    return rows;
}
uint64_t chunk_limit(uint64_t n, uint64_t rows, int P, int G) { return (uint64_t)P * ((n + rows - 1) / rows) + (uint64_t)G; }

hipError_t launch_step(const LloydArgs& g, uint64_t chunks, hipStream_t st) {
    const dim3 grid((unsigned)chunks), block(kTrainThreads);
    if (const int kr = tile_block(g.n, g.P, g.G, g.k, g.dp)) {
        const size_t lds = tile_layout(g.dp, g.kp, tile_vectors(g.dp)).total;
        auto launch = [&](auto kr_c) {
            constexpr int KR = decltype(kr_c)::value;
            if (tile_vectors(g.dp) == 2) hipLaunchKernelGGL((lloyd_tile_kernel<KR, 2, 1>), grid, block, lds, st, g);
            else hipLaunchKernelGGL((lloyd_tile_kernel<KR, 1, 2>), grid, block, lds, st, g);
        };
        switch (kr) {
            case 1: launch(std::integral_constant<int, 1>{}); break;
            case 2: launch(std::integral_constant<int, 2>{}); break;
            case 3: launch(std::integral_constant<int, 3>{}); break;
            case 4: launch(std::integral_constant<int, 4>{}); break;
            case 5: launch(std::integral_constant<int, 5>{}); break;
            case 6: launch(std::integral_constant<int, 6>{}); break;
            case 7: launch(std::integral_constant<int, 7>{}); break;
            case 8: launch(std::integral_constant<int, 8>{}); break;
            default: launch(std::integral_constant<int, 12>{}); break;
        }
        return hipGetLastError();
    }
    const size_t lds = sizeof(uint32_t) * (kTrainThreads / kWave) * (size_t)g.k;
    if (ways_of(g.n, g.P, g.k) > 1) {                        // (at least 128 centroids: a block is 32 of them)
        hipLaunchKernelGGL((lloyd_step_kernel<32, 4>), grid, block, lds, st, g);
        return hipGetLastError();
    }
    switch (centroid_block(g.k)) {
        case 8: hipLaunchKernelGGL((lloyd_step_kernel<8, 1>), grid, block, lds, st, g); break;
        case 16: hipLaunchKernelGGL((lloyd_step_kernel<16, 1>), grid, block, lds, st, g); break;
        case 24: hipLaunchKernelGGL((lloyd_step_kernel<24, 1>), grid, block, lds, st, g); break;
        default: hipLaunchKernelGGL((lloyd_step_kernel<32, 1>), grid, block, lds, st, g); break;
    }
    return hipGetLastError();
}

// Dimensions of a workgroup of lloyd_update_kernel.  100,000 vectors, 64 and 16, us: 32 cells x 64 dimensions 7.2 and 5.2, 96 x 128 9.6 and 8.7,
// 256 x 64 11.3 and 11.9, 512 x 64 11.2 and 17.4; of level 2, smaller workgroups: 256 x 64 4.8 and 4.8, 2,048 x 64 6.1 and 14.8, 4,608 x 128
// 16.4 and 52.6, 12,288 x 64 36.8 and 134.8.
int update_dims(const LloydArgs& g) { return (uint64_t)g.G * (uint64_t)g.k * (uint64_t)((g.dp + 63) / 64) < 256 ? 16 : 64; }

// Lloyd iterations for the groups of g, from start centroids to the result in g.cen / g.cenI.
hipError_t lloyd_run(const LloydArgs& g, const float* parent, uint64_t rows, int iters, uint32_t* chunk_off, uint4* chunks,
                     hipStream_t st) {
    const uint64_t limit = chunk_limit(g.n, rows, g.P, g.G);
    hipLaunchKernelGGL(lloyd_init_kernel, dim3((unsigned)g.G), dim3(kTrainThreads), 0, st, g, parent);
    hipLaunchKernelGGL(chunk_table_kernel, dim3(1), dim3(1024), 0, st, g.range, g.G, (uint32_t)rows, (uint32_t)limit, chunk_off, chunks);
    hipError_t e = hipGetLastError();
    // a group's chunks are split over the wavefronts of a workgroup: sixteen where there are many of them
    const unsigned threads = limit / (unsigned)g.G >= 64 ? 1024 : 256;
    for (int it = 0; it < iters && e == hipSuccess; ++it) {
        e = launch_step(g, limit, st);
        if (e != hipSuccess) break;
        const int dims = update_dims(g);
        const dim3 grid((unsigned)(g.G * g.k), (unsigned)((g.dp + dims - 1) / dims));
        if (dims == 16) hipLaunchKernelGGL(lloyd_update_kernel<16>, grid, dim3(threads), 0, st, g);
        else hipLaunchKernelGGL(lloyd_update_kernel<64>, grid, dim3(threads), 0, st, g);
        e = hipGetLastError();
    }
    return e;
}

// Code points per line by the largest-remainder method, in whole numbers: line q with use[q] of `total`
// votes gets floor(use[q] * n_codes / total), the code points left over go one each to the lines with the
// largest remainders (ties: smaller q).
std::vector<uint32_t> share_out(const std::vector<uint64_t>& use, uint64_t total, uint32_t n_codes) {
    std::vector<uint32_t> alloc(use.size(), 0);
    if (total == 0) return alloc;
    std::vector<std::pair<uint64_t, uint32_t>> rem;        // (remainder, line)
    uint64_t given = 0;
    for (uint32_t q = 0; q < use.size(); ++q) {
        const uint64_t num = use[q] * n_codes;
        alloc[q] = (uint32_t)(num / total);
        given += alloc[q];
        if (num % total) rem.emplace_back(num % total, q);
    }
    std::sort(rem.begin(), rem.end(), [](const auto& l, const auto& r) { return l.first != r.first ? l.first > r.first : l.second < r.second; });
    for (size_t t = 0; given < n_codes && t < rem.size(); ++t, ++given) alloc[rem[t].second]++;
    return alloc;
}

}  // namespace
}  // namespace pqt

extern "C" int pqt_train(const pqt_train_params* tp, const float* vectors, int device, float* C1_out, float* C2_out,
                         uint8_t* tbl_i, uint8_t* tbl_j, float* tbl_lambda, float* cc_out, void* hip_stream) {
    using namespace pqt;
    if (!tp || !vectors || !C1_out || !C2_out || !cc_out) return fail(PQT_EINVAL, "pqt_train: null argument");
    const uint32_t D = tp->D, P = tp->P, k1 = tp->k1, k2 = tp->k2, M = tp->M;
    if (D == 0 || P == 0 || k1 == 0 || k2 == 0 || M == 0 || D % P || D % M || M % P)
        return fail(PQT_EINVAL, "pqt_train: inconsistent sizes D=%u P=%u k1=%u k2=%u M=%u", D, P, k1, k2, M);
    if (!(P == 1 || P == 2 || P == 4)) return fail(PQT_EUNSUPPORTED, "P=%u: only 1, 2 or 4 tree parts", P);
    if (k1 > PQT_MAX_K1 || k2 > PQT_MAX_R || M > 64 || D > 8192)
        return fail(PQT_EUNSUPPORTED, "k1=%u k2=%u M=%u D=%u beyond the kernel limits", k1, k2, M, D);
    if (tp->n == 0 || tp->n >= 0xffffffffull) return fail(PQT_EINVAL, "pqt_train: n=%llu training vectors", (unsigned long long)tp->n);
    if (tp->n_table > tp->n) return fail(PQT_EINVAL, "pqt_train: n_table exceeds n");
    if (tp->n_table > 0 && (!tbl_i || !tbl_j || !tbl_lambda)) return fail(PQT_EINVAL, "pqt_train: null table array");
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev)
        return fail(PQT_EHIP, "GPU %d is not available (%d visible)", device, ndev);
    DeviceGuard guard(device);
    if (!guard.ok) return fail(PQT_EHIP, "cannot select GPU %d", device);
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);

    const uint32_t n = (uint32_t)tp->n;
    const int dp = (int)(D / P), ds = (int)(D / M);
    const uint32_t cells1 = k1, cells2 = k1 * k2;
    const uint32_t npairs = k1 * (k1 - 1) / 2;
    const uint32_t nt = npairs ? (uint32_t)tp->n_table : 0u;
    const size_t nd4 = ((size_t)dp + 3) / 4;
    if (nt) {                                                // (the table serves an index of these sizes)
        std::string why;
        const int rc = pqt_host::check_sizes(D, P, k1, k2, M, 0, 1, 1, 1, PQT_CODES_TABLE, nullptr, why);
        if (rc != PQT_OK) return fail(rc, "%s", why.c_str());
        if (traverse_lds_bytes(D, P, k1, k2, M, 1) > kMaxLds)
            return fail(PQT_EUNSUPPORTED, "pqt_train: D=%u exceeds the LDS budget of the traversal", D);
    }
    LloydArgs l1 = {}, l2 = {};
    l1.X = vectors; l1.n = n; l1.D = (int)D; l1.dp = dp; l1.P = (int)P;
    l1.wide = reinterpret_cast<uintptr_t>(vectors) % 16 == 0 && D % 4 == 0 && dp % 4 == 0;
    l2 = l1;
    l1.G = (int)P; l1.k = (int)k1; l1.kp = padded_centroids(n, (int)P, l1.G, l1.k, dp);
    l2.G = (int)(P * k1); l2.k = (int)k2; l2.kp = padded_centroids(n, (int)P, l2.G, l2.k, dp);
    const uint64_t rows1 = chunk_rows(n, (int)P, l1.G, l1.k, dp), rows2 = chunk_rows(n, (int)P, l2.G, l2.k, dp);
    const uint64_t limit1 = chunk_limit(n, rows1, (int)P, l1.G), limit2 = chunk_limit(n, rows2, (int)P, l2.G);
    // labels are counted in at most 1024 pieces per part
    const uint32_t piece = (uint32_t)(((uint64_t)n + 1024ull * kCellThreads - 1) / (1024ull * kCellThreads) * kCellThreads);
    const uint32_t pieces = (uint32_t)(((uint64_t)n + piece - 1) / piece);
    // lambdas of a line that one workgroup reads; longer lines are cut (into less than 2^20 slices in all)
    const uint32_t slice = (uint32_t)std::max<uint64_t>(16384, (uint64_t)M * nt >> 16);
    // sub-parts whose lambdas are brought together at a time: as many as have 2^27 votes
    const uint32_t batch = nt ? std::min<uint32_t>(M, std::max<uint32_t>(1, (1u << 27) / nt)) : 0u;
    Arena mem;
    double* sums = nullptr;
    uint32_t *counts = nullptr, *label = nullptr, *places = nullptr, *members = nullptr, *chunk_off = nullptr;
    uint4* chunks = nullptr;
    float* dmin = nullptr;
    uint2 *range1 = nullptr, *range2 = nullptr;
    mem.want(&sums, (size_t)std::max(limit1 * k1, limit2 * k2) * dp);
    mem.want(&counts, (size_t)std::max(limit1 * k1, limit2 * k2));
    mem.want(&label, (size_t)P * n);
    mem.want(&places, (size_t)P * k1 * pieces);
    mem.want(&members, (size_t)P * n);
    mem.want(&dmin, (size_t)P * n);
    mem.want(&chunk_off, (size_t)l2.G + 1);
    mem.want(&chunks, (size_t)std::max(limit1, limit2));
    mem.want(&range1, P);
    mem.want(&range2, (size_t)P * k1);
    mem.want(&l1.frozen, P);
    mem.want(&l2.frozen, (size_t)P * k1);
    mem.want(&l1.cen, (size_t)P * cells1 * dp);
    mem.want(&l1.cenI, (size_t)P * nd4 * l1.kp * 4);
    mem.want(&l2.cen, (size_t)P * cells2 * dp);
    mem.want(&l2.cenI, (size_t)P * k1 * nd4 * l2.kp * 4);
    LinePair* pair_dev = nullptr;
    float *c1n_dev = nullptr, *lam_dev = nullptr;
    unsigned long long* keys = nullptr;
    uint32_t *lines_dev = nullptr, *lam_keys = nullptr;
    uint32_t *ranks_dev = nullptr, *bits_dev = nullptr, *digits_dev = nullptr;
    uint4* jobs_dev = nullptr;
    uint2* items_dev = nullptr;
    if (nt) {
        mem.want(&pair_dev, (size_t)M * npairs);
        mem.want(&c1n_dev, (size_t)M * k1);
        mem.want(&keys, (size_t)M * nt);
        mem.want(&lam_keys, (size_t)batch * nt);
        mem.want(&lines_dev, (size_t)M * npairs);
        mem.want(&jobs_dev, (size_t)M * 256);
        mem.want(&ranks_dev, (size_t)M * 256);
        // long lines: a line's slices for every kPicks of its code points, at most
        if (nt > slice) {
            mem.want(&items_dev, (size_t)M * (256 + (256 / kPicks + 1) * (size_t)(nt / slice)));
            mem.want(&bits_dev, (size_t)M * 256);
            mem.want(&digits_dev, (size_t)M * 256 * 256);
        }
        mem.want(&lam_dev, (size_t)M * 256);
    }
    HIP_TRY(mem.allocate());
    l1.range = range1; l2.range = range2;
    l2.members = members;
    l1.chunk_off = l2.chunk_off = chunk_off;
    l1.chunks = l2.chunks = chunks;
    l1.sums = l2.sums = sums; l1.counts = l2.counts = counts; l1.dmin = l2.dmin = dmin;
    std::vector<float> C1, C2, cc;
    std::vector<LinePair> pair_host;
    std::vector<uint32_t> first, ranks;
    std::vector<uint4> jobs, long_jobs;
    std::vector<uint2> items;
    std::vector<float> lam;
    try {
        C1.resize((size_t)P * k1 * dp);
        C2.resize((size_t)P * cells2 * dp);
        cc.resize((size_t)M * k1 * k1);
        pair_host.resize(nt ? (size_t)M * npairs : 0);
        first.resize(nt ? (size_t)M * npairs : 0);
        jobs.reserve(nt ? (size_t)M * 256 : 0);
        long_jobs.reserve(nt > slice ? (size_t)M * 256 : 0);
        items.reserve(nt > slice ? (size_t)M * (256 + (256 / kPicks + 1) * (size_t)(nt / slice)) : 0);
        ranks.resize(nt ? (size_t)M * 256 : 0, 0u);
        lam.resize(nt ? (size_t)M * 256 : 0);
    } catch (const std::bad_alloc&) {
        return fail(PQT_ENOMEM, "host allocation failed");
    }

    const unsigned tb = 256;
    hipLaunchKernelGGL(whole_range_kernel, dim3(1), dim3(kWave), 0, st, n, (int)P, range1);
    // ---- level 1: one group per tree part, k1 centroids ------------------------------------------------
    HIP_TRY(lloyd_run(l1, nullptr, rows1, (int)tp->iters, chunk_off, chunks, st));
    // ---- the cells of the finished quantisers: members in ascending vector order --------------------------
    LloydArgs cells = l1;
    cells.label = label;
    HIP_TRY(launch_step(cells, limit1, st));
    const dim3 by_piece(pieces, P);
    hipLaunchKernelGGL(cell_counts_kernel, by_piece, dim3(kCellThreads), sizeof(uint32_t) * k1, st, label, (uint64_t)n, (int)k1, piece, places);
    hipLaunchKernelGGL(cell_places_kernel, dim3(P), dim3(kCellThreads), 0, st, places, n, (int)k1, pieces, range2);
    hipLaunchKernelGGL(cell_members_kernel, by_piece, dim3(kCellThreads), sizeof(uint32_t) * (kCellWaves + 1) * k1, st, label, (uint64_t)n,
                       (int)k1, piece, places, members);
    HIP_TRY(hipGetLastError());
    // ---- level 2: the cells of all parts, k2 centroids each, trained side by side ---------------------------
    HIP_TRY(lloyd_run(l2, l1.cen, rows2, (int)tp->iters, chunk_off, chunks, st));
    HIP_TRY(hipMemcpyAsync(C1.data(), l1.cen, C1.size() * sizeof(float), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipMemcpyAsync(C2.data(), l2.cen, C2.size() * sizeof(float), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    memcpy(C1_out, C1.data(), C1.size() * sizeof(float));
    memcpy(C2_out, C2.data(), C2.size() * sizeof(float));

    // ---- distances between the level-1 centroids of every sub-part (Sec. 3.3: the table of c^2) -----------
    const size_t per = M / P;
    for (size_t m = 0; m < M; ++m) {
        const size_t p = m / per, lo = m * ds - p * dp;
        for (size_t s = 0; s < k1; ++s)
            for (size_t t = 0; t < k1; ++t) {
                double acc = 0.0;
                for (int d = 0; d < ds; ++d) {
                    const double diff = (double)C1[(p * k1 + s) * dp + lo + d] - (double)C1[(p * k1 + t) * dp + lo + d];
                    acc += diff * diff;
                }
                cc[(m * k1 + s) * k1 + t] = (float)acc;
            }
    }
    memcpy(cc_out, cc.data(), cc.size() * sizeof(float));
    if (tbl_i) memset(tbl_i, 0, (size_t)M * 256);
    if (tbl_j) memset(tbl_j, 0, (size_t)M * 256);
    if (tbl_lambda) memset(tbl_lambda, 0, (size_t)M * 256 * sizeof(float));
    if (nt == 0) return PQT_OK;

    // ---- line table: one vote per sub-vector of the first n_table, by the kernel that encodes vectors ------------------
    {
        size_t e = 0;
        for (size_t m = 0; m < M; ++m)
            for (uint32_t i = 0; i < k1; ++i)
                for (uint32_t j = i + 1; j < k1; ++j) pair_host[e++] = LinePair{i | (j << 16), cc[(m * k1 + i) * k1 + j]};
    }
    HIP_TRY(hipMemcpyAsync(pair_dev, pair_host.data(), pair_host.size() * sizeof(LinePair), hipMemcpyHostToDevice, st));
    PlaceArgs pa = {};
    pa.x = vectors; pa.n = nt;
    pa.D = (int)D; pa.P = (int)P; pa.k1 = (int)k1; pa.k2 = (int)k2; pa.M = (int)M;
    pa.C1 = l1.cen; pa.c1n = c1n_dev; pa.pairs = pair_dev; pa.npairs = (int)npairs; pa.keys = keys;
    HIP_TRY(launch_subpart_norms(l1.cen, (int)D, (int)P, (int)k1, (int)M, c1n_dev, st));
    HIP_TRY(launch_votes(pa, st));
    const dim3 by_vote((unsigned)(((uint64_t)nt + kCellThreads - 1) / kCellThreads), M);
    const size_t nlines = (size_t)M * npairs, lines_lds = npairs <= kLdsLines ? sizeof(uint32_t) * npairs : 0;
    hipLaunchKernelGGL(clear_counts_kernel, dim3((unsigned)((nlines + tb - 1) / tb)), dim3(tb), 0, st, lines_dev, nlines);
    hipLaunchKernelGGL(vote_counts_kernel, by_vote, dim3(kCellThreads), lines_lds, st, keys, nt, (int)npairs, lines_dev);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(first.data(), lines_dev, nlines * sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    // a line's code points sit at the (t + 1/2) / alloc quantiles of its lambdas; lines in pair order and
    // lambdas ascending, so the entries come out ordered by (i, j, lambda)
    for (uint32_t m = 0; m < M; ++m) {
        uint32_t* fm = first.data() + (size_t)m * npairs;    // counts, then first places
        std::vector<uint64_t> use(fm, fm + npairs);
        uint64_t total = 0;
        for (uint32_t q = 0; q < npairs; ++q) {
            fm[q] = (uint32_t)total;
            total += use[q];
        }
        if (total == 0) continue;                            // (no sub-vector has a usable line)
        const std::vector<uint32_t> alloc = share_out(use, total, 256);
        uint32_t c = m * 256;                                // (the shares of a sub-part add up to 256)
        for (uint32_t q = 0; q < npairs; ++q)
            for (uint32_t t = 0; t < alloc[q]; ++t, ++c) {
                const uint64_t pos = ((2ull * t + 1ull) * use[q]) / (2ull * alloc[q]);
                ranks[c] = (uint32_t)std::min(pos, use[q] - 1);
                auto& list = use[q] > slice ? long_jobs : jobs;
                if (t % kPicks == 0) {
                    if (use[q] > slice)
                        for (uint32_t part = 0; (uint64_t)part * slice < use[q]; ++part) items.push_back(make_uint2((uint32_t)long_jobs.size(), part));
                    list.push_back(make_uint4(fm[q], (uint32_t)use[q], c, 0u));
                }
                list.back().w++;
                tbl_i[c] = (uint8_t)pair_host[(size_t)m * npairs + q].ij;
                tbl_j[c] = (uint8_t)(pair_host[(size_t)m * npairs + q].ij >> 16);
            }
    }
    HIP_TRY(hipMemcpyAsync(lines_dev, first.data(), nlines * sizeof(uint32_t), hipMemcpyHostToDevice, st));
    HIP_TRY(hipMemcpyAsync(ranks_dev, ranks.data(), ranks.size() * sizeof(uint32_t), hipMemcpyHostToDevice, st));
    const size_t short_jobs = jobs.size();
    jobs.insert(jobs.end(), long_jobs.begin(), long_jobs.end());
    if (!jobs.empty()) HIP_TRY(hipMemcpyAsync(jobs_dev, jobs.data(), jobs.size() * sizeof(uint4), hipMemcpyHostToDevice, st));
    if (!long_jobs.empty()) {
        const size_t digits = (size_t)M * 256 * 256;
        HIP_TRY(hipMemcpyAsync(items_dev, items.data(), items.size() * sizeof(uint2), hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(clear_counts_kernel, dim3((unsigned)((digits + tb - 1) / tb)), dim3(tb), 0, st, digits_dev, digits);
    }
    size_t job = 0, long_job = short_jobs, item = 0;
    for (uint32_t m0 = 0; m0 < M; m0 += batch) {
        const uint32_t m1 = std::min(M, m0 + batch);
        hipLaunchKernelGGL(vote_groups_kernel, dim3(by_vote.x, m1 - m0), dim3(kCellThreads), lines_lds, st, keys + (size_t)m0 * nt, nt, (int)npairs,
                           lines_dev + (size_t)m0 * npairs, lam_keys);
        const size_t j0 = job, l0 = long_job, i0 = item;
        while (job < short_jobs && jobs[job].z < m1 * 256) ++job;
        while (long_job < jobs.size() && jobs[long_job].z < m1 * 256) ++long_job;
        while (item < items.size() && items[item].x < long_job - short_jobs) ++item;
        if (job > j0)
            hipLaunchKernelGGL(pick_lambdas_kernel, dim3((unsigned)(job - j0)), dim3(kPickThreads), 0, st, lam_keys, nt, m0, jobs_dev + j0, ranks_dev,
                               lam_dev);
        for (int shift = 24; shift >= 0 && long_job > l0; shift -= 8) {
            hipLaunchKernelGGL(slice_digits_kernel, dim3((unsigned)(item - i0)), dim3(1024), 0, st, lam_keys, nt, m0, jobs_dev + short_jobs,
                               items_dev + i0, slice, shift, bits_dev, digits_dev);
            hipLaunchKernelGGL(next_digits_kernel, dim3((unsigned)(long_job - l0)), dim3(256), 0, st, jobs_dev + l0, shift, ranks_dev, bits_dev,
                               digits_dev, lam_dev);
        }
    }
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(lam.data(), lam_dev, lam.size() * sizeof(float), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    for (const uint4& job : jobs) memcpy(tbl_lambda + job.z, lam.data() + job.z, job.w * sizeof(float));
    return PQT_OK;
}
