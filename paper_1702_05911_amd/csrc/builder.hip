// Offline phase on the GPU (Sec. 3.1 "bin map", Sec. 3.3 "Offline computation", Sec. 4): given the
// trained codebooks and the line-code table, database vectors are streamed through; each gets its bin slot
// and its line-quantisation code (place.hip), and at the end
// the ids are ordered by (slot, id) -- a stable radix sort, so ids ascend inside a slot -- the
// pointer array is read off the sorted slots, and the codes are permuted into the same order.
#include <hipcub/hipcub.hpp>

#include <new>

#include "pqt_device.hpp"
#include "pqt_index.hpp"

using pqt_host::DeviceGuard;
using pqt_host::fail;

namespace pqt {

__global__ void iota_kernel(uint32_t* out, uint64_t n) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (uint32_t)i;
}

// Pointer array: offsets[h] = first place of the sorted slots that is not below h (Sec. 4: the prefix sum of the slot
// histogram, without the histogram, whose additions to full slots queue up); also the number of slots that hold a vector.
// A workgroup has `per` * 256 consecutive slots and looks their places up between those of its first and last.
constexpr int kOffsetThreads = 256;
__global__ __launch_bounds__(kOffsetThreads) void offsets_kernel(const uint32_t* sorted, uint32_t n, uint64_t H, int per, uint32_t* offsets,
                                                                 unsigned long long* nonempty) {
    __shared__ uint32_t ends[2];
    const int tid = threadIdx.x;
    const uint64_t h0 = (uint64_t)blockIdx.x * kOffsetThreads * per, h1 = h0 + (uint64_t)kOffsetThreads * per;
    auto place = [&](uint64_t h, uint32_t lo, uint32_t hi) {
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2;
            if (sorted[mid] < h) lo = mid + 1; else hi = mid;
        }
        return lo;
    };
    if (tid < 2) ends[tid] = place(tid ? h1 : h0, 0, n);
    __syncthreads();
    const uint32_t lo = ends[0], hi = ends[1];
    uint32_t filled = 0;
    for (int u = 0; u < per; ++u) {
        const uint64_t h = h0 + (uint64_t)u * kOffsetThreads + tid;
        if (h > H) break;
        const uint32_t at = place(h, lo, hi);
        offsets[h] = at;
        filled += at < hi && sorted[at] == h ? 1u : 0u;
    }
    for (int off = 32; off > 0; off >>= 1) filled += (uint32_t)__shfl_xor((int)filled, off, kWave);
    if ((tid & (kWave - 1)) == 0 && filled) atomicAdd(nonempty, (unsigned long long)filled);
}

// codes_out[i] = codes_in[order[i]], one thread per row of M bytes
__global__ void permute_codes_kernel(const uint8_t* in, const uint32_t* order, uint64_t n, int M, uint8_t* out) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint8_t* src = in + (size_t)order[i] * M;
    uint8_t* dst = out + (size_t)i * M;
    if (M % 4 == 0) {
        for (int j = 0; j < M / 4; ++j) reinterpret_cast<uint32_t*>(dst)[j] = reinterpret_cast<const uint32_t*>(src)[j];
    } else {
        for (int j = 0; j < M; ++j) dst[j] = src[j];
    }
}

}  // namespace pqt

struct pqt_builder {
    pqt_index* ix = nullptr;       // codebooks and tables on the GPU; receives the lists at the end
    uint64_t N = 0, added = 0;
    uint32_t* slots = nullptr;     // N
    uint8_t* codes = nullptr;      // N x M, in id order
};

extern "C" {

int pqt_builder_create(const pqt_index_arrays* params, int device, pqt_builder** out) {
    if (!params || !out) return fail(PQT_EINVAL, "pqt_builder_create: null argument");
    *out = nullptr;
    if (params->N == 0) return fail(PQT_EINVAL, "pqt_builder_create: N = 0");
    pqt_index* ix = nullptr;
    int rc = pqt_host::make_index_without_lists(params, device, &ix);
    if (rc) return rc;
    if (params->N >= 0xffffffffull) {
        pqt_index_free(ix);
        return fail(PQT_EUNSUPPORTED, "N=%llu: 32-bit ids only", (unsigned long long)params->N);
    }
    pqt_builder* b = new (std::nothrow) pqt_builder();
    if (!b) {
        pqt_index_free(ix);
        return fail(PQT_ENOMEM, "host allocation failed");
    }
    b->ix = ix;
    b->N = params->N;
    DeviceGuard guard(device);
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&b->slots), sizeof(uint32_t) * b->N);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&b->codes), (size_t)b->N * ix->code_bytes());
    if (e != hipSuccess) {
        pqt_builder_free(b);
        return fail(e == hipErrorOutOfMemory ? PQT_ENOMEM : PQT_EHIP, "pqt_builder_create: %s", hipGetErrorString(e));
    }
    *out = b;
    return PQT_OK;
}

void pqt_builder_free(pqt_builder* b) {
    if (!b) return;
    if (b->ix) {
        DeviceGuard guard(b->ix->device);
        (void)hipFree(b->slots); (void)hipFree(b->codes);
        pqt_index_free(b->ix);
    }
    delete b;
}

int pqt_builder_add(pqt_builder* b, const float* vectors, int64_t n, void* hip_stream) {
    if (!b || !b->ix) return fail(PQT_EINVAL, "pqt_builder_add: null builder");
    if (n < 0 || b->added + (uint64_t)n > b->N)
        return fail(PQT_EINVAL, "pqt_builder_add: %lld more vectors after %llu exceed N=%llu", (long long)n,
                    (unsigned long long)b->added, (unsigned long long)b->N);
    if (n == 0) return PQT_OK;
    if (!vectors) return fail(PQT_EINVAL, "pqt_builder_add: null vectors");
    pqt_index* ix = b->ix;
    DeviceGuard guard(ix->device);
    if (!guard.ok) return fail(PQT_EHIP, "cannot select GPU %d", ix->device);
    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    if (pqt::traverse_lds_bytes(ix->D, ix->P, ix->k1, ix->k2, ix->M, 1) > pqt::kMaxLds)
        return fail(PQT_EUNSUPPORTED, "pqt_builder_add: D=%u exceeds the LDS budget of the traversal", ix->D);
    pqt::PlaceArgs pa = {};
    pa.x = vectors; pa.n = n;
    pa.D = (int)ix->D; pa.P = (int)ix->P; pa.k1 = (int)ix->k1; pa.k2 = (int)ix->k2; pa.M = (int)ix->M;
    pa.C1 = ix->C1; pa.c1n = ix->c1n; pa.C2 = ix->C2; pa.C2t = ix->C2t;
    pa.table = ix->table; pa.npairs = (int)(ix->k1 * (ix->k1 - 1) / 2);
    pa.k1k2 = ix->k1 * ix->k2; pa.H = ix->H;
    pa.codes = b->codes + (size_t)b->added * ix->code_bytes();
    pa.slots = b->slots + b->added;
    HIP_TRY(pqt::launch_place(pa, ix->code_format == PQT_CODES_PAIR_LAMBDA, stream));
    b->added += (uint64_t)n;
    return PQT_OK;
}

int pqt_builder_finish(pqt_builder* b, pqt_index** out) {
    if (!b || !b->ix || !out) return fail(PQT_EINVAL, "pqt_builder_finish: null argument");
    *out = nullptr;
    if (b->added != b->N)
        return fail(PQT_EINVAL, "pqt_builder_finish: %llu of N=%llu vectors added", (unsigned long long)b->added,
                    (unsigned long long)b->N);
    pqt_index* ix = b->ix;
    DeviceGuard guard(ix->device);
    if (!guard.ok) return fail(PQT_EHIP, "cannot select GPU %d", ix->device);
    HIP_TRY(hipDeviceSynchronize());
    const uint64_t N = b->N;
    uint32_t *ids_in = nullptr, *ids_out = nullptr, *slots_out = nullptr, *offsets = nullptr;
    uint8_t* codes_out = nullptr;
    unsigned long long *nonempty_dev = nullptr, nonempty = 0;
    void* temp = nullptr;
    auto cleanup = [&]() {
        (void)hipFree(ids_in); (void)hipFree(slots_out); (void)hipFree(nonempty_dev); (void)hipFree(temp);
    };
#define BUILD_TRY(expr)                                                                                          \
    do {                                                                                                         \
        hipError_t e_ = (expr);                                                                                  \
        if (e_ != hipSuccess) {                                                                                  \
            cleanup();                                                                                           \
            (void)hipFree(ids_out); (void)hipFree(offsets); (void)hipFree(codes_out);                            \
            return fail(e_ == hipErrorOutOfMemory ? PQT_ENOMEM : PQT_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
        }                                                                                                        \
    } while (0)
    BUILD_TRY(hipMalloc(reinterpret_cast<void**>(&ids_in), sizeof(uint32_t) * N));
    BUILD_TRY(hipMalloc(reinterpret_cast<void**>(&ids_out), sizeof(uint32_t) * N));
    BUILD_TRY(hipMalloc(reinterpret_cast<void**>(&slots_out), sizeof(uint32_t) * N));
    const unsigned tb = 256;
    const unsigned nb = (unsigned)((N + tb - 1) / tb);
    hipLaunchKernelGGL(pqt::iota_kernel, dim3(nb), dim3(tb), 0, 0, ids_in, N);
    // ids by (slot, id): stable sort on the slot
    int end_bit = 1;
    while (end_bit < 32 && (1ull << end_bit) < ix->H) ++end_bit;
    size_t temp_bytes = 0;
    BUILD_TRY(hipcub::DeviceRadixSort::SortPairs(nullptr, temp_bytes, b->slots, slots_out, ids_in, ids_out, N, 0, end_bit));
    BUILD_TRY(hipMalloc(&temp, temp_bytes ? temp_bytes : 1));
    BUILD_TRY(hipcub::DeviceRadixSort::SortPairs(temp, temp_bytes, b->slots, slots_out, ids_in, ids_out, N, 0, end_bit));
    (void)hipFree(temp);
    temp = nullptr;
    // pointer array; about 4096 workgroups of up to 32 slots a thread
    BUILD_TRY(hipMalloc(reinterpret_cast<void**>(&offsets), sizeof(uint32_t) * ((size_t)ix->H + 1)));
    BUILD_TRY(hipMalloc(reinterpret_cast<void**>(&nonempty_dev), sizeof(unsigned long long)));
    BUILD_TRY(hipMemset(nonempty_dev, 0, sizeof(unsigned long long)));
    const uint64_t want = (ix->H + 1) / (4096ull * pqt::kOffsetThreads);
    const int per = want < 1 ? 1 : (want > 32 ? 32 : (int)want);
    const uint64_t span = (uint64_t)pqt::kOffsetThreads * per;
    hipLaunchKernelGGL(pqt::offsets_kernel, dim3((unsigned)((ix->H + 1 + span - 1) / span)), dim3(pqt::kOffsetThreads), 0, 0, slots_out,
                       (uint32_t)N, (uint64_t)ix->H, per, offsets, nonempty_dev);
    BUILD_TRY(hipGetLastError());
    // codes in the order of the ids
    BUILD_TRY(hipMalloc(reinterpret_cast<void**>(&codes_out), (size_t)N * ix->code_bytes()));
    hipLaunchKernelGGL(pqt::permute_codes_kernel, dim3(nb), dim3(tb), 0, 0, b->codes, ids_out, N, (int)ix->code_bytes(),
                       codes_out);
    BUILD_TRY(hipGetLastError());
    BUILD_TRY(hipMemcpy(&nonempty, nonempty_dev, sizeof(nonempty), hipMemcpyDeviceToHost));
    BUILD_TRY(hipDeviceSynchronize());
#undef BUILD_TRY
    cleanup();
    (void)hipFree(ix->offsets); (void)hipFree(ix->ids); (void)hipFree(ix->codes);
    ix->offsets = offsets;
    ix->ids = ids_out;
    ix->codes = codes_out;
    ix->bytes_index += (uint64_t)N * (4 + ix->code_bytes());
    ix->N = N;
    ix->nonempty_slots = nonempty;
    (void)hipFree(b->slots); (void)hipFree(b->codes);
    b->slots = nullptr; b->codes = nullptr;
    *out = ix;
    b->ix = nullptr;                      // the index now belongs to the caller
    return PQT_OK;
}

}  // extern "C"
