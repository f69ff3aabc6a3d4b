// Exact squared distance of a query to database rows, 16 bytes of a row per lane and step: shared by the exact
// re-ranking of a short list and the brute-force search.
#pragma once
#include "pqt_device.hpp"

namespace pqt {

// One 16-byte piece of a row: kElems elements; adds their squared differences to acc in
// ascending dimension.  y points at the query's elements of the same dimensions (LDS).
template <typename Elem>
struct Piece;
template <>
struct Piece<float> {
    static constexpr int kElems = 4;
    static __device__ __forceinline__ float add(uint4 x, int piece, const float* y, float acc) {
        const float4 v = reinterpret_cast<const float4*>(y)[piece];
        float d = v.x - __uint_as_float(x.x);
        acc = fmaf(d, d, acc);
        d = v.y - __uint_as_float(x.y);
        acc = fmaf(d, d, acc);
        d = v.z - __uint_as_float(x.z);
        acc = fmaf(d, d, acc);
        d = v.w - __uint_as_float(x.w);
        return fmaf(d, d, acc);
    }
};
template <>
struct Piece<uint8_t> {
    static constexpr int kElems = 16;
    static __device__ __forceinline__ float add(uint4 x, int piece, const float* y, float acc) {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float4 v = reinterpret_cast<const float4*>(y)[piece * 4 + j];
            float d = v.x - (float)(w[j] & 0xffu);
            acc = fmaf(d, d, acc);
            d = v.y - (float)((w[j] >> 8) & 0xffu);
            acc = fmaf(d, d, acc);
            d = v.z - (float)((w[j] >> 16) & 0xffu);
            acc = fmaf(d, d, acc);
            d = v.w - (float)(w[j] >> 24);
            acc = fmaf(d, d, acc);
        }
        return acc;
    }
};

// lanes that share a row: a power of two, at most 64, one 16-byte piece per lane and step if possible
__device__ __forceinline__ int lanes_per_row(int npieces) {
    int lpr = 1;
    while (lpr < kWave && lpr < npieces) lpr <<= 1;
    return lpr;
}

// ||y - x||^2 of the row every group of lpr lanes has (row < 0: none, 0 is returned): squared differences are
// summed per lane in ascending dimension, then across the group by a fixed xor tree -- the same order in every
// lane, so the result does not depend on scheduling.  l = lane within its group.
template <typename Elem>
__device__ __forceinline__ float row_distance(const Elem* X, int64_t row, int D, const float* y, int lpr, int l) {
    const int npieces = D / Piece<Elem>::kElems;
    float acc = 0.0f;
    if (row >= 0) {
        const Elem* x = X + (size_t)row * D;
        for (int piece = l; piece < npieces; piece += lpr)
            acc = Piece<Elem>::add(reinterpret_cast<const uint4*>(x)[piece], piece, y, acc);
    }
    for (int off = 1; off < lpr; off <<= 1) acc += __shfl_xor(acc, off, kWave);
    return acc;
}

}  // namespace pqt
