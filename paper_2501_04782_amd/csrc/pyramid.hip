// Gaussian pyramid of target frames for the spatial hierarchy (Sec. 3.3):
// each level is the previous one blurred by the separable 5-tap binomial
// filter [1 4 6 4 1] / 16 and decimated by 2 (even rows and columns kept),
// borders mirrored without repeating the edge sample.
//
// HBM-bound when large.  A thread computes a column strip of ROWS output rows,
// two outputs wide: every input row is filtered horizontally once (the five most
// recent results stay in registers for the vertical filter) instead of once
// per output row that reads it, and one 16-byte load brings the four samples
// under the two outputs; the three samples beside them are reads of the
// neighbouring lanes' cache lines.  Sums run in the order of the direct 5 x 5
// form (rows inside, columns outside), so the values are the same bit for bit.
// 50 960x540 frames, 4 levels: 340 us with one output per thread (25
// four-byte loads each), 105 us now; reading and writing every level
// once at the copy rate would take 82 us.  Narrow planes without 16-byte rows
// keep one output per thread (k_pyr_narrow).
#include "gv_internal.h"

namespace gv {

// Rows per strip: 8 read an input row 1.2 times; 2 (1.75 times) give four times
// the threads, for levels that would not fill the chip with strips of 8 (below
// PYR_FEW threads: 16 waves on each of 256 CUs; 5 levels of a 1920x1080 frame
// 33 us with one output per thread, 27 us so), and for heights that would leave
// more than three tenths of a strip of 8 empty (65,536 planes of 20x20: 59 us
// in strips of 8, 54 of 2; of 4x4, 1,048,576 planes: 169 and 56).
constexpr int64_t PYR_FEW = 256 * 16 * 64;

// i mirrored into [0, n) without repeating the edges.
__device__ __forceinline__ int mirror_index(int i, int n) {
    if (n < 3) return n == 1 ? 0 : i & 1;  // period 2 (n - 1)
    if (i < 0) i = -i;
    return i >= n ? 2 * (n - 1) - i : i;
}

// How a thread reads the samples 2x - 2 .. 2x + 4 under its outputs x and
// x + 1: rows that start on 16-byte boundaries (W % 4 == 0; x is even); any
// other row, in vector loads of 4-byte alignment, where all seven lie inside
// it; the first and last pairs of such a row, sample by sample (39 frames of
// 739x738, 4 levels: 277 us at first, 182 us in strips with four-byte loads
// throughout, 101 us with these).
enum Reads { ALIGNED, INSIDE, EDGE };
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));

// Horizontal filter at the outputs x and x + 1 of one input row.
template <Reads R>
__device__ __forceinline__ float2 filter_row(const float* __restrict__ row, int x, int W) {
    float v[7];
    if (R == ALIGNED) {
        const float4 m = *reinterpret_cast<const float4*>(row + 2 * x);
        const bool right = 2 * x + 4 < W;
        const float2 l = *reinterpret_cast<const float2*>(row + (x > 0 ? 2 * x - 2 : 0));
        const float r = row[right ? 2 * x + 4 : 0];
        v[0] = x > 0 ? l.x : m.z;
        v[1] = x > 0 ? l.y : m.y;
        v[2] = m.x;
        v[3] = m.y;
        v[4] = m.z;
        v[5] = m.w;
        v[6] = right ? r : m.z;
    } else if (R == INSIDE) {
        const float4u l = *reinterpret_cast<const float4u*>(row + 2 * x - 2);
        const float2u r = *reinterpret_cast<const float2u*>(row + 2 * x + 2);
        v[0] = l.x;
        v[1] = l.y;
        v[2] = l.z;
        v[3] = l.w;
        v[4] = r.x;
        v[5] = r.y;
        v[6] = row[2 * x + 4];
    } else {
        // the second output may lie past the row: its samples are clamped
        // into the mirror's reach and its value is not stored
#pragma unroll
        for (int d = 0; d < 7; ++d) v[d] = row[mirror_index(min(2 * x + d - 2, W + 1), W)];
    }
    const float k[5] = {0.0625f, 0.25f, 0.375f, 0.25f, 0.0625f};
    float2 h = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int d = 0; d < 5; ++d) {
        h.x += k[d] * v[d];
        h.y += k[d] * v[d + 2];
    }
    return h;
}

template <Reads R, int ROWS>
__device__ __forceinline__ void filter_strip(const float* __restrict__ src, float* __restrict__ dst, int x, int y0,
                                             int H, int W, int Ho, int Wo) {
    auto at = [&](int y) { return filter_row<R>(src + static_cast<int64_t>(mirror_index(y, H)) * W, x, W); };
    const float k[5] = {0.0625f, 0.25f, 0.375f, 0.25f, 0.0625f};
    float2 h[5];
    h[0] = at(2 * y0 - 2);
    h[1] = at(2 * y0 - 1);
    h[2] = at(2 * y0);
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const int y = min(y0 + j, Ho - 1);  // rows past the end repeat the last one's reads and are not stored
        h[3] = at(2 * y + 1);
        h[4] = at(2 * y + 2);
        float2 acc = make_float2(0.0f, 0.0f);
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            acc.x += k[d] * h[d].x;
            acc.y += k[d] * h[d].y;
        }
        if (y0 + j < Ho) {
            if (R == ALIGNED) {
                *reinterpret_cast<float2*>(dst) = acc;
            } else {
                dst[0] = acc.x;
                if (x + 1 < Wo) dst[1] = acc.y;
            }
        }
        dst += Wo;
        h[0] = h[2];
        h[1] = h[3];
        h[2] = h[4];
    }
}

// I: index type (32 bits while the threads fit).
template <bool VEC, int ROWS, typename I>
__global__ __launch_bounds__(256) void k_pyr_reduce(const float* __restrict__ in, float* __restrict__ out, I threads,
                                                    int H, int W, int Ho, int Wo) {
    const I i = static_cast<I>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= threads) return;
    const I pairs = static_cast<I>((Wo + 1) >> 1), strips = static_cast<I>((Ho + ROWS - 1) / ROWS);
    const I r = i / pairs;
    const int x = 2 * static_cast<int>(i - r * pairs);
    const I p = r / strips;
    const int y0 = static_cast<int>(r - p * strips) * ROWS;
    const float* src = in + static_cast<int64_t>(p) * H * W;
    float* dst = out + static_cast<int64_t>(p) * Ho * Wo + static_cast<int64_t>(y0) * Wo + x;
    if (VEC) filter_strip<ALIGNED, ROWS>(src, dst, x, y0, H, W, Ho, Wo);
    else if (x >= 2 && 2 * x + 4 < W) filter_strip<INSIDE, ROWS>(src, dst, x, y0, H, W, Ho, Wo);
    else filter_strip<EDGE, ROWS>(src, dst, x, y0, H, W, Ho, Wo);
}

// The remaining levels of small planes in one launch: a workgroup per plane
// keeps a level in LDS while it computes the next, so levels of a few
// microseconds do not each wait for a launch.  One thread per output, the sums
// in the same order.  Taken when at least two levels remain and the plane has
// at most PYR_TAIL samples.  64 frames of 206x139, 6 levels: 37 us with a
// launch per level, 24 us with two launches.  And for at most PYR_TAIL_PLANES
// planes, four to each workgroup that the chip holds at a time: small planes
// leave most of a workgroup idle (2,048 planes of 32x32, 4 launches 27 us
// against 19; 4,096 27 against 36; 1,048,576 planes of 8x8 154 us against
// 4,442), and a launch holds fewer than 2^32 threads.
constexpr int PYR_TAIL = 8192;
constexpr int64_t PYR_TAIL_PLANES = 2048;
constexpr int TAIL_WG = 1024;

__global__ __launch_bounds__(TAIL_WG) void k_pyr_tail(const float* __restrict__ in, float* __restrict__ out,
                                                  int64_t planes, int h, int w, int levels) {
    __shared__ float A[PYR_TAIL], B[PYR_TAIL / 2 + 1];  // a row of PYR_TAIL samples leaves half
    const int64_t p = blockIdx.x;
    for (int i = threadIdx.x; i < h * w; i += TAIL_WG) A[i] = in[p * h * w + i];
    const float k[5] = {0.0625f, 0.25f, 0.375f, 0.25f, 0.0625f};
    float *src = A, *dst = B;
    for (int l = 0; l < levels; ++l) {
        __syncthreads();
        const int ho = (h + 1) / 2, wo = (w + 1) / 2;
        float* o = out + p * ho * wo;
        for (int i = threadIdx.x; i < ho * wo; i += TAIL_WG) {
            const int y = i / wo, x = i - y * wo;
            int xs[5];
#pragma unroll
            for (int d = 0; d < 5; ++d) xs[d] = mirror_index(2 * x + d - 2, w);
            float acc = 0.0f;
#pragma unroll
            for (int dy = 0; dy < 5; ++dy) {
                const float* row = src + mirror_index(2 * y + dy - 2, h) * w;
                float r = 0.0f;
#pragma unroll
                for (int dx = 0; dx < 5; ++dx) r += k[dx] * row[xs[dx]];
                acc += k[dy] * r;
            }
            o[i] = dst[i] = acc;
        }
        out += planes * ho * wo;
        h = ho;
        w = wo;
        float* t = src;
        src = dst;
        dst = t;
    }
}

// Rows of up to PYR_NARROW outputs that take no 16-byte loads: one thread per
// output, so that a wave reads neighbouring samples.  A wave of strips reads as
// many distant rows as it has strips side by side: 65,536 planes of 64x1 88 us
// against 41, of 300x11 1,274 against 987, 1,048,576 of 14x14 1,057 against
// 915; beyond (64x17) 356 us in strips against 479.
constexpr int PYR_NARROW = 8;

__global__ __launch_bounds__(256) void k_pyr_narrow(const float* __restrict__ in, float* __restrict__ out,
                                                    int64_t outputs, int H, int W, int Ho, int Wo) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= outputs) return;
    const int64_t per = static_cast<int64_t>(Ho) * Wo;
    const int64_t p = i / per;
    const int r = static_cast<int>(i - p * per);
    const int y = r / Wo, x = r - y * Wo;
    const float k[5] = {0.0625f, 0.25f, 0.375f, 0.25f, 0.0625f};
    const float* src = in + p * static_cast<int64_t>(H) * W;
    int xs[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) xs[d] = mirror_index(2 * x + d - 2, W);
    float acc = 0.0f;
#pragma unroll
    for (int dy = 0; dy < 5; ++dy) {
        const float* row = src + static_cast<int64_t>(mirror_index(2 * y + dy - 2, H)) * W;
        float h = 0.0f;
#pragma unroll
        for (int dx = 0; dx < 5; ++dx) h += k[dx] * row[xs[dx]];
        acc += k[dy] * h;
    }
    out[i] = acc;
}

template <bool VEC, int ROWS>
static void launch_strips(const float* src, float* dst, int64_t planes, int h, int w, int ho, int wo, hipStream_t st) {
    const int64_t threads = planes * ((ho + ROWS - 1) / ROWS) * ((wo + 1) / 2);
    const dim3 grid(static_cast<uint32_t>((threads + 255) / 256)), block(256);
    if (threads > 0x7fffff00LL)
        hipLaunchKernelGGL((k_pyr_reduce<VEC, ROWS, uint64_t>), grid, block, 0, st, src, dst,
                           static_cast<uint64_t>(threads), h, w, ho, wo);
    else
        hipLaunchKernelGGL((k_pyr_reduce<VEC, ROWS, uint32_t>), grid, block, 0, st, src, dst,
                           static_cast<uint32_t>(threads), h, w, ho, wo);
}

static hipError_t launch_pyr_reduce(const float* src, float* dst, int64_t planes, int h, int w, int ho, int wo,
                                    hipStream_t st) {
    // 16-byte loads and 8-byte stores need rows that start on those
    // boundaries; other widths (one level in two of a ragged frame) take
    // 4-byte accesses
    const bool vec = w % 4 == 0 && (reinterpret_cast<uintptr_t>(src) & 15u) == 0u &&
                     (reinterpret_cast<uintptr_t>(dst) & 7u) == 0u;
    if (!vec && wo <= PYR_NARROW) {
        const int64_t n = planes * static_cast<int64_t>(ho) * wo;
        hipLaunchKernelGGL(k_pyr_narrow, dim3(static_cast<uint32_t>((n + 255) / 256)), dim3(256), 0, st, src, dst, n, h, w,
                           ho, wo);
        return hipGetLastError();
    }
    const int strips = (ho + 7) / 8;
    const bool few = 80 * strips > 13 * ho || planes * strips * ((wo + 1) / 2) < PYR_FEW;
    if (vec && few) launch_strips<true, 2>(src, dst, planes, h, w, ho, wo, st);
    else if (vec) launch_strips<true, 8>(src, dst, planes, h, w, ho, wo, st);
    else if (few) launch_strips<false, 2>(src, dst, planes, h, w, ho, wo, st);
    else launch_strips<false, 8>(src, dst, planes, h, w, ho, wo, st);
    return hipGetLastError();
}

}  // namespace gv

using namespace gv;

static bool pyramid_args_ok(int64_t planes, int32_t height, int32_t width, int32_t levels) {
    return planes >= 1 && height >= 1 && width >= 1 && height <= 65536 && width <= 65536 && levels >= 1 &&
           levels <= 16 && planes * static_cast<int64_t>(height) * width <= (int64_t(1) << 40);
}

extern "C" gv_status gv_pyramid_floats(int64_t planes, int32_t height, int32_t width, int32_t levels,
                                       int64_t* out_count) {
    if (!out_count || !pyramid_args_ok(planes, height, width, levels)) return GV_ERR_INVALID_ARG;
    int64_t total = 0;
    int h = height, w = width;
    for (int l = 1; l < levels; ++l) {
        h = (h + 1) / 2;
        w = (w + 1) / 2;
        total += planes * static_cast<int64_t>(h) * w;
    }
    *out_count = total;
    return GV_OK;
}

extern "C" gv_status gv_gaussian_pyramid(const float* images, int64_t planes, int32_t height, int32_t width,
                                         int32_t levels, float* out, void* stream) {
    if (!images || !pyramid_args_ok(planes, height, width, levels) || (levels > 1 && !out))
        return GV_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const float* src = images;
    float* dst = out;
    int h = height, w = width;
    for (int l = 1; l < levels; ++l) {
        if (levels - l >= 2 && static_cast<int64_t>(h) * w <= PYR_TAIL && planes <= PYR_TAIL_PLANES) {
            hipLaunchKernelGGL(k_pyr_tail, dim3(static_cast<uint32_t>(planes)), dim3(TAIL_WG), 0, st, src, dst, planes, h, w,
                               levels - l);
            return hipGetLastError() == hipSuccess ? GV_OK : GV_ERR_HIP;
        }
        const int ho = (h + 1) / 2, wo = (w + 1) / 2;
        const int64_t n = planes * static_cast<int64_t>(ho) * wo;
        const hipError_t e = launch_pyr_reduce(src, dst, planes, h, w, ho, wo, st);
        if (e != hipSuccess) return GV_ERR_HIP;
        src = dst;
        dst += n;
        h = ho;
        w = wo;
    }
    return GV_OK;
}
