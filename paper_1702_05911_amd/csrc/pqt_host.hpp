// Host-only parts of the library that touch no GPU: the index-file reader, the validation of index
// arrays, and the builder of the fixed traversal-order tables.  Plain C++ (no HIP header), so that this
// code also compiles into a CPU test program under the address and undefined-behaviour sanitizers.
#pragma once
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/pqt.h"

namespace pqt_host {

// First 64 bytes of the 256-byte file header.
struct FileHeader {
    char magic[8];
    uint32_t version, D, P, k1, k2, M;
    uint64_t N, H;
    uint32_t T, C, offset_bits, code_format;
};
static_assert(sizeof(FileHeader) == 64, "header prefix is 64 bytes");

// An index file in host memory (layout: see pqt_index_load in pqt.h).
struct IndexFile {
    uint32_t D = 0, P = 0, k1 = 0, k2 = 0, M = 0, T = 0, C = 0, code_format = 0;
    uint64_t N = 0, H = 0;
    std::vector<float> C1, C2, lam, cc;
    std::vector<uint8_t> ti, tj, codes;
    std::vector<uint32_t> offsets, ids;
};

// Reads and checks the header, then the nine sections.  Returns PQT_OK or PQT_EIO / PQT_EFORMAT /
// PQT_EUNSUPPORTED / PQT_ENOMEM with a message in err.  Nothing is allocated before the sizes in the
// header have passed check_sizes and are consistent with the length of the file.
int read_index_file(const char* path, IndexFile& out, std::string& err);

// Sizes and limits of an index (everything that can be said without looking at the arrays).
int check_sizes(uint32_t D, uint32_t P, uint32_t k1, uint32_t k2, uint32_t M, uint64_t N, uint64_t H, uint32_t T, uint32_t C,
                uint32_t code_format, bool* hashed, std::string& err);

// The arrays that live in host memory: the pointer array spans the ids and is monotone (also counts the
// slots that hold a vector), table entries name centroids below k1, and -- when the codes are in host
// memory (codes != null) and hold (pair, lambda) tuples -- every pair byte names a pair.
int check_arrays(uint32_t k1, uint32_t M, uint64_t N, uint64_t H, uint32_t code_format, const uint32_t* offsets,
                 const uint8_t* tbl_i, const uint8_t* tbl_j, const uint8_t* codes, uint64_t* nonempty, std::string& err);

// The fixed anisotropic traversal order (Sec. 3.2 "Bin Proposal Heuristic"): ten pre-computed orders of the
// rank pairs, one per slope 1.08^k, k = -5..4.  table receives kSlopes x Tn entries r1 << 16 | r2 with
// Tn = min(T, R^2) (returned); thr the nine boundaries 1.08^(j - 5.5), j = 1..9, between neighbouring slopes.
constexpr int kSlopes = 10;
int make_static_order(int R, int T, std::vector<uint32_t>& table, float thr[kSlopes - 1]);

// How far the brute-force filter's sum for a vector x may lie from ||x||^2 / 2 - q.x (brute_force.hip): dot * ||q|| ||x|| + norm *
// ||x||^2 + kBruteUnderflow.  elem_bytes: 1 for byte vectors, 4 for floats.
//   * Cutting.  bf16 has eight significant bits: of x = s 2^e, 1 <= s < 2, a first piece leaves at most 2^(e-8), which a second
//     piece leaves at most 2^(e-17) of.  Floats: the product of two second pieces is dropped, 2^-16 of a product, and
//     both numbers' remainders, 2^-17 each: 2^-15.  Bytes are one piece exactly: the query's remainder, 2^-17.  Times
//     ||q|| ||x|| by Cauchy-Schwarz.
//   * Adding up.  16 products a matrix instruction and the running sum are taken to be added one by one in any order, every
//     addition off by at most 2^-23 of its result (rounded or truncated): nothing is assumed about how an instruction adds
//     inside.  A partial sum is at most ||q|| ||x|| + ||x||^2 / 2.
//   * The norm's own sum: at most 24 + D / 64 additions a lane and across lanes, and four roundings of what it starts from.
//   * The centre: both floats lose 2^-24 of themselves when it is subtracted.
//   * Underflow.  The matrix cores may take numbers below 2^-126, the smallest normal one, for zero: a second piece, a product
//     or a sum.  At most six such losses per dimension of up to 8,192 (2^-110), and pieces times the other vector, which
//     the next power of two and the relative terms cover.
// 3 % on top for the terms of higher order and the rounding of the norms.
//   * Halves (brute_error_half): eleven significant bits, so either number loses up to 2^-11 of itself, 2^-10 of a product; one
//     product instead of three is added up.  Both are scaled so that the query's norm and the largest vector's lie in 2^14 ..
//     2^15, and what then lies below 2^-14, the smallest normal half, may be taken for zero: sqrt(D) 2^-14 of such numbers against the
//     other's norm, 2^-28 sqrt(D) ||q|| X for either, X the largest norm of all (flush ||q|| X).
//     The first chunk's values are those of pieces, and what the list may hold is bounded for both kinds at once: dot and dot + 2 norm,
//     the parts of the window (keep_up_to), are no smaller than the pieces', whose three products weigh more than
//     the shorter numbers from about 2,000 dimensions on.
struct BruteError {
    float dot, norm, flush;
};
constexpr float kBruteUnderflow = 0x1p-109f;
BruteError brute_error(int elem_bytes, int D);
BruteError brute_error_half(int D);

// Is a small batch faster in one launch, a query a workgroup, than in three?  A workgroup of its own does by itself what the traversal
// kernel's sixteen queries share: the level-1 products with D k1 codebook values, one row of sixteen used; and the values of a child come
// one after the other, which weighs about as sixteen centroids more.  Up to 16 queries the traversal's tile is as good as empty,
// above 256 two or four workgroups have a compute unit; many candidates, one part, or lists of more than 64 entries, whose
// ranking is long, leave more to gain.  Three launches and one, us (lists of up to 64, two parts, 1,000 candidates unless given):
//   D = 960, k1 = 64       one query 53 and 60, 12 60 and 61, 256 76 and 68, 300 82 and 94, 700 91 and 129, 1,024 100 and 161
//   D = 960, k1 = 16       one query 35 and 35 (M = 16: 34 and 35), 4 37 and 35, 300 51 and 48, 1,024 64 and 69 (four parts 300 75 and 67; 4,096 candidates 1,024 82 and 75)
//   D = 512, k1 = 64       one query 44 and 45, 300 65 and 63, 700 78 and 86, 1,024 87 and 101 (four parts 300 77 and 82)
//   D = 512, k1 = 16       one query 30 and 28, 1,024 55 and 54;   D = 1,536, k1 = 16 one query 41 and 43, 300 63 and 61, 1,024 77 and 91
//   D = 1,536, k1 = 64     256 96 and 88, four parts 16 78 and 89
//   D = 192, k1 = 64       one query 56 and 33, 1,024 76 and 64;   D = 320, k1 = 32  1,024 72 and 58
//   lists of 128: D = 960, k1 = 16 1,024 104 and 81, k1 = 64 300 106 and 97;  one part: D = 960, k1 = 16 1,024 86 and 64, k1 = 64 113 and 146
bool one_launch_pays(uint32_t D, uint32_t P, uint32_t k1, int R, uint32_t C, int64_t nq);

// number of pairs (a, b), a < nA, b < nB, with (a+1)(b+1) <= Tn
long region_size(int nA, int nB, int Tn);

}  // namespace pqt_host
