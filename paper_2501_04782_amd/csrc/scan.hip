// Exclusive prefix sum of the tiles' intersection counts: the tile ranges.  The
// grand total is kept in 64 bits so that an intersection count beyond 2^32 is
// detected as an overflow instead of wrapping.
//
// Bound by launches and latency, not bytes (8 bytes per tile).  Up to
// SCAN_ONE tiles one workgroup scans them all (one launch; a 960x540 frame has
// 2,040); above, each workgroup scans SCAN_TILE counts and a second launch adds
// what lies before, every workgroup summing the earlier workgroups' totals
// itself.  With the clears in one kernel and the two last reductions of the
// adjoint in another, a 128x128 step went from 17 launches to 9 (the sort has
// since taken a second) and from 143 to 129 us, one 960x540 frame of 100k
// Gaussians from 359 to 328 us.
#include "gv_internal.h"

namespace gv {

constexpr int SCAN_THREADS = 1024;
constexpr int SCAN_ITEMS = 4;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;  // 4096 counts per workgroup
constexpr int64_t SCAN_ONE = 4 * SCAN_TILE;

// Exclusive scan of x across the threads of the workgroup; returns the prefix
// and the workgroup's total.
__device__ __forceinline__ unsigned long long block_exclusive_scan(unsigned long long x, unsigned long long& total) {
    __shared__ unsigned long long wsum[SCAN_THREADS / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned long long inc = x;
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    unsigned long long before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < SCAN_THREADS / 64; ++k) {
        const unsigned long long v = wsum[k];
        if (k < w) before += v;
        all += v;
    }
    total = all;
    __syncthreads();
    return before + inc - x;
}

// The workgroup's SCAN_TILE counts from `base` on: their exclusive prefix sums
// plus `before` go to out.  Returns their total.
__device__ __forceinline__ unsigned long long scan_tile(const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                                                        int64_t base, int64_t count, unsigned long long before) {
    const int64_t i = base + threadIdx.x * SCAN_ITEMS;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (i + SCAN_ITEMS <= count) {  // regions of the workspace start on 256-byte boundaries
        v = *reinterpret_cast<const uint4*>(in + i);
    } else {
        if (i < count) v.x = in[i];
        if (i + 1 < count) v.y = in[i + 1];
        if (i + 2 < count) v.z = in[i + 2];
    }
    unsigned long long total;
    const unsigned long long sum = static_cast<unsigned long long>(v.x) + v.y + v.z + v.w;
    const uint32_t run = static_cast<uint32_t>(before + block_exclusive_scan(sum, total));
    const uint4 o = make_uint4(run, run + v.x, run + v.x + v.y, run + v.x + v.y + v.z);
    if (i + SCAN_ITEMS <= count) {
        *reinterpret_cast<uint4*>(out + i) = o;
    } else {
        if (i < count) out[i] = o.x;
        if (i + 1 < count) out[i + 1] = o.y;
        if (i + 2 < count) out[i + 2] = o.z;
    }
    return total;
}

// The grand total: the end of the last range and the status words.
__device__ __forceinline__ void finish_scan(const Args& a, int64_t count, unsigned long long total) {
    a.toff[count] = static_cast<uint32_t>(total);
    a.status[ST_K_LO] = static_cast<uint32_t>(total);
    a.status[ST_K_HI] = static_cast<uint32_t>(total >> 32);
    if (total > static_cast<uint64_t>(a.k_cap)) a.status[ST_OVERFLOW] = 1u;
    if (a.total_out) __hip_atomic_store(a.total_out, total + 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_one(Args a, int64_t count) {
    unsigned long long run = 0;
    for (int64_t base = 0; base < count; base += SCAN_TILE) run += scan_tile(a.tcnt, a.toff, base, count, run);
    if (threadIdx.x == 0) finish_scan(a, count, run);
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_local(Args a, int64_t count, unsigned long long* __restrict__ sums) {
    const unsigned long long total =
        scan_tile(a.tcnt, a.toff, static_cast<int64_t>(blockIdx.x) * SCAN_TILE, count, 0ull);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_add(Args a, int64_t count,
                                                           const unsigned long long* __restrict__ sums) {
    const int64_t b = blockIdx.x;
    unsigned long long mine = 0, before;
    for (int64_t k = threadIdx.x; k < b; k += SCAN_THREADS) mine += sums[k];
    block_exclusive_scan(mine, before);
    const int64_t base = b * SCAN_TILE;
    for (int k = threadIdx.x; k < SCAN_TILE; k += SCAN_THREADS)
        if (base + k < count) a.toff[base + k] += static_cast<uint32_t>(before);
    if (b == gridDim.x - 1 && threadIdx.x == 0) finish_scan(a, count, before + sums[b]);
}

int64_t scan_blocks(int64_t count) { return (count + SCAN_TILE - 1) / SCAN_TILE; }

// Scan of a.tcnt into a.toff; tmp holds scan_blocks(frames * tiles) 64-bit
// values.
hipError_t launch_tile_scan(const Args& a, unsigned long long* tmp, hipStream_t stream) {
    const int64_t count = static_cast<int64_t>(a.frames) * a.tiles;
    const dim3 block(SCAN_THREADS);
    if (count <= SCAN_ONE) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), block, 0, stream, a, count);
        return hipGetLastError();
    }
    const dim3 grid(static_cast<uint32_t>(scan_blocks(count)));
    hipLaunchKernelGGL(k_scan_local, grid, block, 0, stream, a, count, tmp);
    hipLaunchKernelGGL(k_scan_add, grid, block, 0, stream, a, count, tmp);
    return hipGetLastError();
}

}  // namespace gv
