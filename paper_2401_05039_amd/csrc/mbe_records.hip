// Canonical order of enumerated bicliques (device side).
//
// The search writes records [|A|, |B|, A..., B...] in whatever order its waves finish.  The
// canonical output sorts each side ascending and the records by A lexicographically; A
// determines B (B = N(A)), so the order is total.

#include <rocprim/device/device_merge_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "mbe_internal.h"

namespace mbe {

namespace {

// Ascending sort of a[0, n) in place by 16 lanes (l: the lane's number among them): a bitonic network
// whose comparisons all put the smaller entry first, so entries past n, as if the largest, stay.
__device__ void sort_long_side(int32_t *a, int n, int l) {
    auto order = [&](int i, int j) {
        if (j >= n) return;
        const int32_t x = __hip_atomic_load(a + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const int32_t y = __hip_atomic_load(a + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (x > y) {
            __hip_atomic_store(a + i, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_store(a + j, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    for (int64_t k = 2; k < 2 * (int64_t)n; k <<= 1) {  // blocks of k entries
        // i and its mirror in the block, then pairs of ever smaller distance
        for (int64_t h = k >> 1; h > 0; h >>= 1) {
            for (int64_t t = l;; t += 16) {
                const int64_t i = (t / h) * 2 * h + t % h;
                if (i >= n) break;
                const int64_t j = 2 * h == k ? i + k - 1 - 2 * (t % h) : i + h;
                if (j < n) order((int)i, (int)j);
            }
            __threadfence_block();
        }
    }
}

// Ascending sort of a[0, n), distinct entries, by 16 lanes (l: the lane's number among them).  Up to
// 64 entries are held 4 per lane and placed by rank, one shuffle per entry and lane; longer sides are
// sorted in memory.
__device__ __forceinline__ void sort_side(int32_t *a, int n, int l) {
    if (n > 64) {
        sort_long_side(a, n, l);
        return;
    }
    int32_t e[4];
    int rank[4] = {0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) e[q] = 16 * q + l < n ? a[16 * q + l] : 0x7FFFFFFF;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (16 * q >= n) break;
        for (int j = 0; j < 16 && 16 * q + j < n; ++j) {
            const int32_t x = __shfl(e[q], j, 16);
#pragma unroll
            for (int t = 0; t < 4; ++t) rank[t] += x < e[t] ? 1 : 0;
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (16 * q + l < n) a[rank[q]] = e[q];
}

// Sorts the sides of every record and writes the sort keys of all index slots (those that hold no
// record come last).  16 lanes per record: a thread per record, with its sides in memory, took 0.8 ms for
// 516,620 records of 8 ints, this 0.15 ms.  keys == NULL: none are written.
__global__ void sort_sides_kernel(int32_t *rec, const unsigned long long *offs, unsigned long long n, RecordKey *keys) {
    const int l = (int)(threadIdx.x & 15u);
    const unsigned long long stride = ((unsigned long long)gridDim.x * blockDim.x) >> 4;
    for (unsigned long long i = ((unsigned long long)blockIdx.x * blockDim.x + threadIdx.x) >> 4; i < n; i += stride) {
        const unsigned long long off = offs[i];
        if (off == kNoRecord) {
            if (l == 0 && keys) keys[i] = RecordKey{~0ull, kNoRecord};
            continue;
        }
        int32_t *r = rec + off;
        const int na = r[0], nb = r[1];
        sort_side(r + 2, na, l);
        sort_side(r + 2 + na, nb, l);
        __threadfence_block();
        if (l == 0 && keys) {
            const unsigned int a0 = (unsigned int)r[2], a1 = na > 1 ? (unsigned int)r[3] + 1u : 0u;
            keys[i] = RecordKey{((unsigned long long)a0 << 32) | a1, off};
        }
    }
}

__device__ __forceinline__ unsigned long long offset_of(const RecordKey &k) { return k.off; }
__device__ __forceinline__ unsigned long long offset_of(unsigned long long k) { return k; }

// By the first two vertices of A, then by the whole of A.
struct RecordLess {
    const int32_t *rec;
    __device__ bool operator()(const RecordKey &x, const RecordKey &y) const {
        if (x.head != y.head) return x.head < y.head;
        if (x.off == kNoRecord || y.off == kNoRecord) return false;  // (only both)
        return after(x.off, y.off, 2);
    }
    __device__ bool operator()(unsigned long long x, unsigned long long y) const { return after(x, y, 0); }
    // the same from the i-th vertex of A on
    __device__ bool after(unsigned long long x, unsigned long long y, int i) const {
        const int32_t *a = rec + x;
        const int32_t *b = rec + y;
        const int na = a[0], nb = b[0];
        const int n = na < nb ? na : nb;
        for (; i < n; ++i) {
            const int32_t p = a[2 + i], q = b[2 + i];
            if (p != q) return p < q;
        }
        return na < nb;
    }
};

template <typename K>
__global__ void lengths_kernel(const int32_t *rec, const K *keys, unsigned long long n,
                               unsigned long long *lens) {
    const unsigned long long stride = (unsigned long long)gridDim.x * blockDim.x;
    for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int32_t *r = rec + offset_of(keys[i]);
        lens[i] = 2ull + (unsigned long long)r[0] + (unsigned long long)r[1];
    }
}

// one wave per record: copy it to its place in the output
template <typename K>
__global__ void gather_kernel(const int32_t *rec, const K *keys, const unsigned long long *dst,
                              unsigned long long n, int32_t *out) {
    const int lane = (int)__lane_id();
    const unsigned long long wave = ((unsigned long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const unsigned long long nwaves = ((unsigned long long)gridDim.x * blockDim.x) >> 6;
    for (unsigned long long i = wave; i < n; i += nwaves) {
        const int32_t *r = rec + offset_of(keys[i]);
        const unsigned long long len = 2ull + (unsigned long long)r[0] + (unsigned long long)r[1];
        int32_t *o = out + dst[i];
        for (unsigned long long q = lane; q < len; q += 64) o[q] = r[q];
    }
}

int grid_for(unsigned long long n, int block) {
    unsigned long long g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > 8192) g = 8192;
    return (int)g;
}

// Sorts keys (n_slots of them, those of the n_rec records first) into sorted and writes the records to
// out in that order; offs receives their places.  With temp == NULL only *temp_bytes is set.
template <typename K>
hipError_t sort_and_gather(const int32_t *rec, unsigned long long *offs, K *keys, K *sorted, unsigned long long n_slots,
                           unsigned long long n_rec, unsigned long long *lens, int32_t *out, void *temp,
                           size_t *temp_bytes, hipStream_t s) {
    const RecordLess less{rec};
    size_t t_sort = 0, t_scan = 0;
    hipError_t e = rocprim::merge_sort(nullptr, t_sort, keys, sorted, (size_t)n_slots, less, s);
    if (e != hipSuccess) return e;
    e = rocprim::exclusive_scan(nullptr, t_scan, lens, offs, 0ull, (size_t)n_rec, rocprim::plus<unsigned long long>(), s);
    if (e != hipSuccess) return e;
    const size_t need = (t_sort > t_scan ? t_sort : t_scan) + 256;
    if (temp == nullptr) {
        *temp_bytes = need;
        return hipSuccess;
    }
    if (*temp_bytes < need) return hipErrorInvalidValue;
    e = rocprim::merge_sort(temp, t_sort, keys, sorted, (size_t)n_slots, less, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(lengths_kernel<K>, dim3(grid_for(n_rec, 256)), dim3(256), 0, s, rec, sorted, n_rec, lens);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    e = rocprim::exclusive_scan(temp, t_scan, lens, offs, 0ull, (size_t)n_rec, rocprim::plus<unsigned long long>(), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(gather_kernel<K>, dim3(grid_for(n_rec * 64, 256)), dim3(256), 0, s, rec, sorted, offs, n_rec, out);
    return hipGetLastError();
}

}  // namespace

// rec: record arena; offs[n_slots]: record start offsets, kNoRecord where an index holds none, n_rec
// others (overwritten); scratch: 2 n_slots RecordKeys, or, with small, n_slots u64 (every index holds
// a record then): the sort compares records by reading both, with a quarter of the scratch; lens:
// n_rec scratch; out: destination (sum of lengths ints).  With temp == NULL only *temp_bytes is set.
hipError_t canonical_records(int32_t *rec, unsigned long long *offs, unsigned long long n_slots,
                             unsigned long long n_rec, void *scratch, bool small, unsigned long long *lens, int32_t *out,
                             void *temp, size_t *temp_bytes, hipStream_t s) {
    RecordKey *keys = small ? nullptr : static_cast<RecordKey *>(scratch);
    if (temp != nullptr) {
        if (n_rec == 0) return hipSuccess;
        hipLaunchKernelGGL(sort_sides_kernel, dim3(grid_for(n_slots * 16, 256)), dim3(256), 0, s, rec, offs, n_slots, keys);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (small)
        return sort_and_gather(rec, offs, offs, static_cast<unsigned long long *>(scratch), n_slots, n_rec, lens, out, temp,
                               temp_bytes, s);
    return sort_and_gather(rec, offs, keys, keys + n_slots, n_slots, n_rec, lens, out, temp, temp_bytes, s);
}

}  // namespace mbe
