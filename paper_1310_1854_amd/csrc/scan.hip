// scan.hip -- exclusive prefix sums of non-negative int32 counts, used for
// CSR row offsets, bucket offsets and per-ray segment offsets.
//
// Three launches and no temporary buffer: tile totals are parked in the
// output at the tile-end positions, scanned in place by one block, and each
// tile then writes its own prefix (the value it rewrites at its end position
// equals what the in-place scan left there, so neighbouring tiles can read
// it concurrently).
#include "vrt_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kItems = 8;
constexpr int kTile = kThreads * kItems;

// Four sums side by side.
struct Int4 {
    int32_t x, y, z, w;
    __device__ Int4 &operator+=(const Int4 &o)
    {
        x += o.x;
        y += o.y;
        z += o.z;
        w += o.w;
        return *this;
    }
    __device__ Int4 operator+(const Int4 &o) const
    {
        Int4 r = *this;
        return r += o;
    }
    __device__ Int4 operator-(const Int4 &o) const
    {
        Int4 r = *this;
        r.x -= o.x;
        r.y -= o.y;
        r.z -= o.z;
        r.w -= o.w;
        return r;
    }
};

template <typename OutT, typename InT>
__device__ __forceinline__ OutT to_sum(const InT &v)
{
    if constexpr (sizeof(InT) == sizeof(int4)) return OutT{v.x, v.y, v.z, v.w};
    else return (OutT)v;
}

template <typename T>
__device__ T block_exclusive_scan(T v, T *lds, T *total)
{
    const int t = threadIdx.x;
    lds[t] = v;
    __syncthreads();
    for (int off = 1; off < blockDim.x; off <<= 1) {
        T add = (t >= off) ? lds[t - off] : T{};
        __syncthreads();
        lds[t] += add;
        __syncthreads();
    }
    T incl = lds[t];
    if (total) *total = lds[blockDim.x - 1];
    __syncthreads();
    return incl - v;
}

template <typename InT, typename OutT>
__global__ void __launch_bounds__(kThreads) k_tile_totals(const InT *__restrict__ counts, int64_t n,
                                                          OutT *__restrict__ out)
{
    __shared__ OutT lds[kThreads];
    const int64_t base = (int64_t)blockIdx.x * kTile;
    OutT s{};
    for (int i = 0; i < kItems; ++i) {
        int64_t idx = base + (int64_t)i * kThreads + threadIdx.x;
        if (idx < n) s += to_sum<OutT>(counts[idx]);
    }
    OutT total;
    block_exclusive_scan<OutT>(s, lds, &total);
    if (threadIdx.x == 0) {
        int64_t end = base + kTile;
        out[end < n ? end : n] = total;
    }
}

template <typename OutT>
__global__ void __launch_bounds__(1024) k_scan_totals(OutT *__restrict__ out, int64_t n, int64_t ntiles)
{
    __shared__ OutT lds[1024];
    OutT carry{};
    for (int64_t c = 0; c < ntiles; c += blockDim.x) {
        int64_t b = c + threadIdx.x;
        int64_t pos = (b + 1) * kTile;
        if (pos > n) pos = n;
        OutT v = (b < ntiles) ? out[pos] : OutT{};
        OutT total;
        OutT ex = block_exclusive_scan<OutT>(v, lds, &total);
        if (b < ntiles) out[pos] = carry + ex + v;
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = OutT{};
}

template <typename InT, typename OutT>
__global__ void __launch_bounds__(kThreads) k_tile_scan(const InT *__restrict__ counts, int64_t n,
                                                        OutT *__restrict__ out)
{
    __shared__ OutT lds[kThreads];
    const int64_t base = (int64_t)blockIdx.x * kTile;
    OutT tile_base = (blockIdx.x == 0) ? OutT{} : out[base];
    // each thread owns kItems consecutive elements
    OutT v[kItems];
    OutT s{};
    for (int i = 0; i < kItems; ++i) {
        int64_t idx = base + (int64_t)threadIdx.x * kItems + i;
        v[i] = (idx < n) ? to_sum<OutT>(counts[idx]) : OutT{};
        s += v[i];
    }
    OutT ex = block_exclusive_scan<OutT>(s, lds, nullptr);
    OutT run = tile_base + ex;
    for (int i = 0; i < kItems; ++i) {
        int64_t idx = base + (int64_t)threadIdx.x * kItems + i;
        run += v[i];
        if (idx < n) out[idx + 1] = run;
    }
}

template <typename InT, typename OutT>
vor_status scan_impl(const InT *counts, int64_t n, OutT *out, hipStream_t st)
{
    if (n < 0 || (!out) || (n > 0 && !counts)) return VOR_EINVAL;
    if (n == 0) {
        OutT zero{};
        return hipMemcpyAsync(out, &zero, sizeof(OutT), hipMemcpyHostToDevice, st) == hipSuccess ? VOR_OK
                                                                                                   : VOR_EDEVICE;
    }
    int64_t ntiles = (n + kTile - 1) / kTile;
    if (ntiles > 0x7fffffff) return VOR_EINVAL;
    hipLaunchKernelGGL((k_tile_totals<InT, OutT>), dim3((unsigned)ntiles), dim3(kThreads), 0, st, counts, n, out);
    hipLaunchKernelGGL(k_scan_totals<OutT>, dim3(1), dim3(1024), 0, st, out, n, ntiles);
    hipLaunchKernelGGL((k_tile_scan<InT, OutT>), dim3((unsigned)ntiles), dim3(kThreads), 0, st, counts, n, out);
    return hipGetLastError() == hipSuccess ? VOR_OK : VOR_EDEVICE;
}

}  // namespace

vor_status vrt_scan_i32_to_i64(const int32_t *counts, int64_t n, int64_t *offsets, hipStream_t st)
{
    return scan_impl<int32_t, int64_t>(counts, n, offsets, st);
}

vor_status vrt_scan_i32_to_i32(const int32_t *counts, int64_t n, int32_t *offsets, hipStream_t st)
{
    return scan_impl<int32_t, int32_t>(counts, n, offsets, st);
}

vor_status vrt_scan_int4(const int4 *counts, int64_t n, int4 *offsets, hipStream_t st)
{
    static_assert(sizeof(Int4) == sizeof(int4), "the sums are stored as int4");
    return scan_impl<int4, Int4>(counts, n, reinterpret_cast<Int4 *>(offsets), st);
}

extern "C" vor_status vor_exclusive_scan(const int32_t *counts, int64_t N, int64_t *offsets, void *stream)
{
    return vrt_scan_i32_to_i64(counts, N, offsets, (hipStream_t)stream);
}
