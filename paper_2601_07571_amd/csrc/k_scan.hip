// k_scan.hip -- exact integer prefix sums (reduce, scan of block totals, scan
// with offsets).  Integer addition is associative, so the result does not depend
// on the blocking.  Used for the triangle-weight scan (uint64, inclusive) and for
// the spatial-bucket offsets of the sample sort (uint32, exclusive).
#include <hip/hip_runtime.h>

#include "gm_internal.h"
#include "gm_lattice.h"

namespace gm {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = 8;
constexpr int kTile = kThreads * kItems;  // elements per block

template <typename T>
__device__ __forceinline__ T wave_inclusive(T v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const T o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    return v;
}

// Exclusive prefix over the block's threads; returns the block total in *total.
template <int Threads = kThreads, typename T>
__device__ __forceinline__ T block_exclusive(T v, T* total)
{
    __shared__ T wsum[Threads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const T inc = wave_inclusive(v);
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < Threads / 64; ++w) {
        if (w < wave) before += wsum[w];
        all += wsum[w];
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

// The kItems elements of a thread from base on (zeros from n on), by 16-byte loads where all of
// them are there (the arrays are aligned to 16 bytes): one element at a time, the scan of 2^24
// buckets took 31 us for the totals and 64 us for the scan, 11 and 24 us this way.
template <typename T>
__device__ __forceinline__ void load_items(const T* in, int64_t base, int64_t n, T (&v)[kItems])
{
    if (base + kItems <= n) {
        uint4* q = reinterpret_cast<uint4*>(v);
#pragma unroll
        for (int i = 0; i < (int)(sizeof(T) * kItems / 16); ++i) q[i] = reinterpret_cast<const uint4*>(in + base)[i];
    } else {
#pragma unroll
        for (int i = 0; i < kItems; ++i) v[i] = base + i < n ? in[base + i] : T(0);
    }
}

// Where a scan's elements come from: an array, or the lattice sampler's point counts of the
// triangles, formed from their areas where they are scanned (no pass that writes them first).
template <typename T>
struct ArrayItems {
    const T* in;
    __device__ __forceinline__ void operator()(int64_t base, int64_t n, T (&v)[kItems]) const { load_items(in, base, n, v); }
};

struct LatticeItems {
    const double* area;
    double k;
    __device__ __forceinline__ void operator()(int64_t base, int64_t n, unsigned long long (&v)[kItems]) const
    {
        alignas(16) double a[kItems];
        load_items(area, base, n, a);
#pragma unroll
        for (int i = 0; i < kItems; ++i) v[i] = base + i < n ? lattice_count(k, a[i]) : 0ull;
    }
};

// the running sums of those elements from `run` on
template <bool Inclusive, typename T>
__device__ __forceinline__ void store_scan(T* out, int64_t base, int64_t n, T (&v)[kItems], T run)
{
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const T x = v[i];
        v[i] = Inclusive ? run + x : run;
        run += x;
    }
    if (base + kItems <= n) {
        const uint4* q = reinterpret_cast<const uint4*>(v);
#pragma unroll
        for (int i = 0; i < (int)(sizeof(T) * kItems / 16); ++i) reinterpret_cast<uint4*>(out + base)[i] = q[i];
    } else {
#pragma unroll
        for (int i = 0; i < kItems; ++i)
            if (base + i < n) out[base + i] = v[i];
    }
}

template <typename T, class Items>
__global__ void __launch_bounds__(kThreads) k_block_totals(Items in, int64_t n, T* __restrict__ totals)
{
    const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;
    alignas(16) T v[kItems];
    in(base, n, v);
    T s = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) s += v[i];
    T tot;
    (void)block_exclusive(s, &tot);
    if (threadIdx.x == 0) totals[blockIdx.x] = tot;
}

// One block scans n elements (out may be in) with a running carry, kItems a thread at a time
// (8,192 totals: 20 us by 256 threads, one each; 5 us this way).
constexpr int kOneThreads = 1024;

template <typename T, bool Inclusive, class Items>
__global__ void __launch_bounds__(kOneThreads) k_scan_one(Items in, T* out, int64_t n)
{
    T carry = 0;
    for (int64_t b0 = 0; b0 < n; b0 += kOneThreads * kItems) {
        const int64_t base = b0 + (int64_t)threadIdx.x * kItems;
        alignas(16) T v[kItems];
        in(base, n, v);
        T s = 0;
#pragma unroll
        for (int i = 0; i < kItems; ++i) s += v[i];
        T tot;
        T run = carry + block_exclusive<kOneThreads>(s, &tot);
        store_scan<Inclusive>(out, base, n, v, run);
        carry += tot;
    }
}

template <typename T, bool Inclusive, class Items>
__global__ void __launch_bounds__(kThreads) k_block_scan(Items in, T* __restrict__ out, int64_t n,
                                                         const T* __restrict__ offsets)
{
    const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;
    alignas(16) T v[kItems];
    in(base, n, v);
    T s = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) s += v[i];
    T tot;
    T run = block_exclusive(s, &tot) + offsets[blockIdx.x];
    store_scan<Inclusive>(out, base, n, v, run);
}

template <typename T, bool Inclusive, class Items>
void scan(Items in, T* out, int64_t n, void* tmp, hipStream_t s)
{
    if (n <= 0) return;
    // one launch where one block takes no longer than three (32,768 elements: 7.4 us; 8 us and
    // two more launches otherwise)
    if (n <= 4 * kOneThreads * kItems) {
        k_scan_one<T, Inclusive, Items><<<1, kOneThreads, 0, s>>>(in, out, n);
        return;
    }
    const int64_t nb = (n + kTile - 1) / kTile;
    T* totals = static_cast<T*>(tmp);
    k_block_totals<T, Items><<<(unsigned)nb, kThreads, 0, s>>>(in, n, totals);
    k_scan_one<T, false><<<1, kOneThreads, 0, s>>>(ArrayItems<T>{totals}, totals, nb);
    k_block_scan<T, Inclusive, Items><<<(unsigned)nb, kThreads, 0, s>>>(in, out, n, totals);
}

}  // namespace

size_t scan_tmp_bytes(int64_t n)
{
    const int64_t nb = (n + kTile - 1) / kTile;
    return (size_t)(nb > 0 ? nb : 1) * sizeof(unsigned long long);
}

void launch_inclusive_scan_u64(const unsigned long long* in, unsigned long long* out, int64_t n, void* tmp,
                               hipStream_t s)
{
    scan<unsigned long long, true>(ArrayItems<unsigned long long>{in}, out, n, tmp, s);
}

void launch_lattice_scan(const double* area, double k, unsigned long long* out, int64_t n, void* tmp, hipStream_t s)
{
    scan<unsigned long long, true>(LatticeItems{area, k}, out, n, tmp, s);
}

void launch_exclusive_scan_u32(const uint32_t* in, uint32_t* out, int64_t n, void* tmp, hipStream_t s)
{
    scan<uint32_t, false>(ArrayItems<uint32_t>{in}, out, n, tmp, s);
}

}  // namespace gm
