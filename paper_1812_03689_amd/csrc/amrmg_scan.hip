// amrmg_scan.hip -- exclusive prefix sums of unsigned integers on the device,
// used by the particle visiting order (the radix sort's tile offsets) and the
// brick-table build (face and update-list offsets).  Up to 16384 values, one
// workgroup in one launch; beyond, two launches:
//   1. every workgroup sums its tile of SCAN_TILE consecutive values;
//   2. every workgroup adds the sums of all tiles before its own (read by the
//      whole workgroup and reduced in LDS) to the exclusive scan of its tile.
// The result is exact (integer arithmetic) and does not depend on the launch
// shape.
#include <hip/hip_runtime.h>

#include "amrmg_kernels.hpp"

namespace amrmg {

constexpr int SCAN_NT = 256, SCAN_PER = 8, SCAN_TILE = SCAN_NT * SCAN_PER;

// inclusive sum over the workgroup's NT threads of one value per thread;
// returns the thread's inclusive prefix and writes the workgroup total to
// *total.  In the wavefront by shuffles, then over the wavefronts' totals
// through LDS: two barriers (doubling steps in LDS take two a step).  lds: NT
// / 64 values.
template <int NT, class V>
__device__ V block_inclusive_scan(V v, V *lds, V *total)
{
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const V add = __shfl_up(v, off, 64);
        if (lane >= off) v += add;
    }
    if (lane == 63) lds[wave] = v;
    __syncthreads();
    V before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const V s = lds[w];
        if (w < wave) before += s;
        all += s;
    }
    if (total) *total = all;
    __syncthreads();
    return before + v;
}

template <class V>
__global__ void __launch_bounds__(SCAN_NT) k_scan_tiles(const V *in, int64_t n, V *tile_sum)
{
    __shared__ V lds[SCAN_NT / 64];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_PER;
    V s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_PER; ++i)
        if (base + i < n) s += in[base + i];
    V total;
    (void)block_inclusive_scan<SCAN_NT>(s, lds, &total);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

template <class V>
__global__ void __launch_bounds__(SCAN_NT) k_scan_apply(const V *in, int64_t n, const V *tile_sum, V *out)
{
    __shared__ V lds[SCAN_NT / 64];
    // the sums of the tiles before this one
    V before = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += SCAN_NT) before += tile_sum[t];
    V prefix;
    (void)block_inclusive_scan<SCAN_NT>(before, lds, &prefix);
    // the tile: each thread scans its SCAN_PER values, the threads' totals are
    // scanned across the workgroup
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_PER;
    V v[SCAN_PER], s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_PER; ++i) {
        v[i] = base + i < n ? in[base + i] : (V)0;
        s += v[i];
    }
    const V incl = block_inclusive_scan<SCAN_NT>(s, lds, (V *)nullptr);
    V run = prefix + incl - s;
#pragma unroll
    for (int i = 0; i < SCAN_PER; ++i) {
        if (base + i < n) out[base + i] = run;
        run += v[i];
    }
}

// Up to SCAN_ONE values: one workgroup of 1024 threads, each scanning PER
// consecutive values (4 or 16, by the count, so that short scans use many
// threads; whole 16-byte loads and stores), the threads' totals scanned
// across the workgroup (one launch instead of two: short scans are
// launch-bound).
constexpr int SCAN_ONE_NT = 1024, SCAN_ONE = SCAN_ONE_NT * 16;

template <class V, int PER>
__global__ void __launch_bounds__(SCAN_ONE_NT) k_scan_one(const V *in, int64_t n, V *out)
{
    __shared__ V lds[SCAN_ONE_NT / 64];
    constexpr int PV = 16 / sizeof(V);
    typedef V Vec __attribute__((ext_vector_type(16 / sizeof(V))));
    const int64_t base = (int64_t)threadIdx.x * PER;
    const bool whole = base + PER <= n;
    V v[PER], s = 0;
    if (whole) {
#pragma unroll
        for (int i = 0; i < PER / PV; ++i) {
            const Vec t = *(const Vec *)(in + base + PV * i);
#pragma unroll
            for (int k = 0; k < PV; ++k) v[PV * i + k] = t[k];
        }
    } else {
#pragma unroll
        for (int i = 0; i < PER; ++i) v[i] = base + i < n ? in[base + i] : (V)0;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) s += v[i];
    V run = block_inclusive_scan<SCAN_ONE_NT>(s, lds, (V *)nullptr) - s;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const V t = v[i];
        v[i] = run;
        run += t;
    }
    if (whole) {
#pragma unroll
        for (int i = 0; i < PER / PV; ++i) {
            Vec t;
#pragma unroll
            for (int k = 0; k < PV; ++k) t[k] = v[PV * i + k];
            *(Vec *)(out + base + PV * i) = t;
        }
    } else {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (base + i < n) out[base + i] = v[i];
    }
}

template <class V>
size_t scan_temp_bytes(int64_t n)
{
    return sizeof(V) * (size_t)((n + SCAN_TILE - 1) / SCAN_TILE + 1);
}

template <class V>
hipError_t exclusive_scan(hipStream_t st, const V *in, V *out, int64_t n, void *temp, size_t temp_bytes)
{
    if (n <= 0) return hipSuccess;
    if (n <= SCAN_ONE) {
        if (((uintptr_t)in | (uintptr_t)out) & 15) return hipErrorInvalidValue;  // 16-byte accesses
        if (n <= SCAN_ONE_NT * 4)
            hipLaunchKernelGGL((k_scan_one<V, 4>), dim3(1), dim3(SCAN_ONE_NT), 0, st, in, n, out);
        else
            hipLaunchKernelGGL((k_scan_one<V, 16>), dim3(1), dim3(SCAN_ONE_NT), 0, st, in, n, out);
        return hipGetLastError();
    }
    if (!temp || temp_bytes < scan_temp_bytes<V>(n)) return hipErrorInvalidValue;
    const int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (tiles > INT32_MAX) return hipErrorInvalidValue;
    V *sums = (V *)temp;
    hipLaunchKernelGGL((k_scan_tiles<V>), dim3((unsigned)tiles), dim3(SCAN_NT), 0, st, in, n, sums);
    hipLaunchKernelGGL((k_scan_apply<V>), dim3((unsigned)tiles), dim3(SCAN_NT), 0, st, in, n, sums, out);
    return hipGetLastError();
}

template size_t scan_temp_bytes<uint32_t>(int64_t);
template size_t scan_temp_bytes<uint64_t>(int64_t);
template hipError_t exclusive_scan<uint32_t>(hipStream_t, const uint32_t *, uint32_t *, int64_t, void *, size_t);
template hipError_t exclusive_scan<uint64_t>(hipStream_t, const uint64_t *, uint64_t *, int64_t, void *, size_t);

}  // namespace amrmg
