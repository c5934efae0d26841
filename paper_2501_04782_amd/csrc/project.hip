// EWA projection of every (frame, Gaussian) pair and the two binning passes
// (count, then scatter of (depth, index) keys into per-tile buckets).
//
// The projection runs in FP64: on CDNA4 the FP64 vector rate equals the
// non-packed FP32 rate, the stage streams 56 bytes per Gaussian from HBM, and
// FP64 keeps the rounded records (centre, conic, depth key) as close to the
// exact values as their storage format allows.  Only the per-pixel loop of the
// compositing kernels runs in FP32.
#include <algorithm>

#include "gv_internal.h"

namespace gv {

// First kernel of a forward: the frame-independent shape of every Gaussian of
// a static scene (no dynamics; once per call instead of once per frame),
// and in the same launch the words the later kernels count in or mark: the
// status, the tiles' counts and next positions, and the adjoint's marks (the
// entries a tile's adjoint writes are fixed by its forward, so one clear here
// serves every adjoint of this forward).  A single 128x128 frame spent a tenth
// of its step in the separate clears.
template <typename T>
__global__ __launch_bounds__(256) void k_begin(Args a, bool shapes, int64_t ft, int64_t marks) {
    const int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (g < ST_WORDS) a.status[g] = 0u;
    if (g < ft) a.tcnt[g] = a.tcur[g] = 0u;
    if (g < marks) a.pused[g] = 0u;
    if (!shapes || g >= a.n) return;
    const int64_t n = a.n;
    double raw[14];
    for (int k = 0; k < 3; ++k) raw[k] = 0.0;
    for (int k = 0; k < 3; ++k) raw[3 + k] = load_param<T>(a.log_scales, k * n + g);
    for (int k = 0; k < 4; ++k) raw[6 + k] = load_param<T>(a.quats, k * n + g);
    raw[10] = load_param<T>(a.opacity_logits, g);
    for (int k = 0; k < 3; ++k) raw[11 + k] = load_param<T>(a.colors, k * n + g);
    bool fin = true;
    for (int k = 3; k < 14; ++k) fin = fin && isfinite(raw[k]);
    if (a.sh_degree > 0) fin = sh_finite<T>(a, g) && fin;
    ShapeD S;
    ProjD P;
    const bool ok = fin && shape_from_params(raw, P);
    for (int k = 0; k < 6; ++k) S.Sig[k] = ok ? P.Sig[k] : 0.0;
    S.o = ok ? P.o : 0.0;
    S.fin = fin ? 1u : 0u;
    S.qn_ok = ok ? 1u : 0u;
    a.shapes[g] = S;
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t value, int64_t count) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < count) p[i] = value;
}

// Tile range [t0, t1] along one axis whose pixel-centre span meets [lo, hi].
__device__ __forceinline__ bool tile_span(double lo, double hi, int n_tiles, int& t0, int& t1) {
    double a = ceil((lo - (TILE - 0.5)) / TILE);
    double b = floor((hi - 0.5) / TILE);
    a = fmax(a, 0.0);
    b = fmin(b, static_cast<double>(n_tiles - 1));
    if (!(a <= b)) return false;
    t0 = static_cast<int>(a);
    t1 = static_cast<int>(b);
    return true;
}

// A projected Gaussian's binning data: its ellipse (centre, rounded conic
// and the edge-minimiser slopes of ellipse_meets_box_r) and its tile
// rectangle (tx0, ty0, width rw, height rh).
struct BinShape {
    double u, v, a, b, c, rbc, rba;
    int tx0, ty0, rw, rh;
};

// Project Gaussian g in frame f: write its record, tile rectangle and colour,
// and return true with its binning shape if it can reach a pixel (visible,
// opacity at least 1/255, non-empty tile rectangle).  Frame 0 also writes
// the per-Gaussian colour/opacity table shared by all frames.
template <bool DYN, bool SH, typename T>
__device__ __forceinline__ bool project_one(const Args& a, int f, int64_t g, const CamD& cam, double t,
                                            const SplineD& basis, BinShape& S) {
    const int64_t i = static_cast<int64_t>(f) * a.n + g;
    if (!SH && f == 0) {
        const double eta = load_param<T>(a.opacity_logits, g);
        ColorOp co;
        co.r = static_cast<float>(load_param<T>(a.colors, g));
        co.g = static_cast<float>(load_param<T>(a.colors, a.n + g));
        co.b = static_cast<float>(load_param<T>(a.colors, 2 * a.n + g));
        co.o = static_cast<float>(1.0 / (1.0 + exp(-eta)));
        a.col4[g] = co;
    }
    ProjD P;
    // without dynamics the shapes are those k_begin computed
    bool vis;
    if constexpr (DYN) vis = project_gaussian<SH, T>(a, g, cam, t, basis, P);
    else vis = project_gaussian_shaped<T>(a, g, cam, t, P);
    if (P.nonfinite) atomicAdd(&a.status[ST_NONFINITE], 1u);
    // o < 1/255 can never pass the per-pixel alpha test (alpha <= o).
    if (!vis || !(P.o >= static_cast<double>(ALPHA_MIN) * (1.0 - 1e-6))) return false;
    Record r;
    r.u = P.u;
    r.v = P.v;
    r.a = static_cast<float>(P.A[0]);
    r.b = static_cast<float>(P.A[1]);
    r.c = static_cast<float>(P.A[2]);
    r.depth = static_cast<float>(P.m[2]);
    // axis-aligned box of the 3-sigma ellipse, padded for the rounded conic
    const double hx = 3.0 * sqrt(P.cov[0]) * (1.0 + 2e-5) + 1e-4;
    const double hy = 3.0 * sqrt(P.cov[2]) * (1.0 + 2e-5) + 1e-4;
    int tx0, tx1, ty0, ty1;
    if (!tile_span(P.u - hx, P.u + hx, a.tiles_x, tx0, tx1) || !tile_span(P.v - hy, P.v + hy, a.tiles_y, ty0, ty1))
        return false;
    a.rec[i] = r;
    a.dkey[i] = r.depth;
    a.rect[i] = make_uint2(static_cast<uint32_t>(tx0) | (static_cast<uint32_t>(tx1) << 16),
                           static_cast<uint32_t>(ty0) | (static_cast<uint32_t>(ty1) << 16));
    if (SH) {  // only now: Gaussians without a tile need no colour
        sh_colour<T>(a, g, cam, P);
        ColorOp co;
        co.r = static_cast<float>(P.col[0]);
        co.g = static_cast<float>(P.col[1]);
        co.b = static_cast<float>(P.col[2]);
        co.o = static_cast<float>(P.o);
        a.col4[i] = co;
    }
    S.u = r.u;
    S.v = r.v;
    S.a = r.a;
    S.b = r.b;
    S.c = r.c;
    S.rbc = -S.b / S.c;
    S.rba = -S.b / S.a;
    S.tx0 = tx0;
    S.ty0 = ty0;
    S.rw = tx1 - tx0 + 1;
    S.rh = ty1 - ty0 + 1;
    return true;
}

// Does the ellipse of S meet tile (tx, ty)?  The one test of both binning
// passes (exact ellipse-box minimum, slack for the fp32 per-pixel test).
__device__ __forceinline__ bool shape_meets_tile(const Args& a, const BinShape& S, int tx, int ty) {
    double x0, x1, y0, y1;
    tile_box(tx, ty, a.width, a.height, x0, x1, y0, y1);
    return ellipse_meets_box_r<double>(S.u, S.v, S.a, S.b, S.c, S.rbc, S.rba, x0, x1, y0, y1, BIN_Q_SLACK);
}

__device__ __forceinline__ BinShape shape_from_record(const Record& r, uint2 rc) {
    BinShape S;
    S.u = r.u;
    S.v = r.v;
    S.a = r.a;
    S.b = r.b;
    S.c = r.c;
    S.rbc = -S.b / S.c;
    S.rba = -S.b / S.a;
    S.tx0 = rc.x & 0xffff;
    S.ty0 = rc.y & 0xffff;
    S.rw = static_cast<int>(rc.x >> 16) - S.tx0 + 1;
    S.rh = static_cast<int>(rc.y >> 16) - S.ty0 + 1;
    return S;
}

// Exclusive prefix sum of x over the wave and the wave total.
__device__ __forceinline__ uint32_t wave_exclusive_scan(uint32_t x, int lane, uint32_t& total) {
    uint32_t incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = static_cast<uint32_t>(__shfl_up(static_cast<int>(incl), d, 64));
        if (lane >= d) incl += t;
    }
    total = static_cast<uint32_t>(__shfl(static_cast<int>(incl), 63, 64));
    return incl - x;
}

// Lane owning work item b0 + lane of a wave whose lanes deal out `cnt` items
// each from exclusive starts `start`: the last lane with items whose start is
// at most the item.  Each owner whose first item falls in [b0, b0 + 64) marks
// that position in `own` (64 slots of the wave, in LDS); an item's owner is
// the mark at or below its position, or, before the first mark, the owner of
// item b0 (the last lane with items starting at or before b0).
__device__ __forceinline__ int chunk_owner(uint32_t* own, uint32_t start, uint32_t cnt, uint32_t b0, int lane) {
    own[lane] = 0u;
    __builtin_amdgcn_wave_barrier();
    if (cnt && start >= b0 && start - b0 < 64u) own[start - b0] = static_cast<uint32_t>(lane) + 1u;
    __builtin_amdgcn_wave_barrier();
    const uint32_t mark = own[lane];
    const uint64_t marks = __ballot(mark != 0u);
    const uint64_t before = __ballot(cnt != 0u && start <= b0);
    const int carry = before ? 63 - __builtin_clzll(before) : 0;
    const uint64_t upto = marks & (lane == 63 ? ~0ull : ((2ull << lane) - 1ull));
    const int src = upto ? 63 - __builtin_clzll(upto) : 0;
    const int m = __shfl(static_cast<int>(mark), src, 64);
    __builtin_amdgcn_wave_barrier();
    return upto ? m - 1 : carry;
}

// Index of the (k+1)-th set bit of m (k < popcount(m)).
__device__ __forceinline__ int kth_set_bit(uint64_t m, uint32_t k) {
    int b = 0;
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
        const uint64_t low = m & ((1ull << w) - 1ull);
        const uint32_t c = static_cast<uint32_t>(__popcll(low));
        if (k >= c) {
            k -= c;
            m >>= w;
            b += w;
        } else {
            m = low;
        }
    }
    return b;
}

// A value equal in every lane, moved to scalar registers.
__device__ __forceinline__ double uniform(double v) {
    const uint64_t b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b >> 32));
    return __longlong_as_double((static_cast<uint64_t>(hi) << 32) | lo);
}

// The workgroup's camera in scalar registers: held in vector registers over the
// rounds it took 24 of them.
__device__ __forceinline__ CamD uniform_camera(const CamD& c) {
    CamD u = c;
    for (int k = 0; k < 9; ++k) u.R[k] = uniform(c.R[k]);
    for (int k = 0; k < 3; ++k) u.t[k] = uniform(c.t[k]);
    u.ok = __builtin_amdgcn_readfirstlane(c.ok ? 1 : 0) != 0;
    return u;
}

// Per-wave LDS staging of the cooperative rectangle walk: the cells of the
// 64 lanes' tile rectangles are dealt out one per lane and step, so a wave
// takes (total cells) / 64 steps instead of its largest rectangle.
struct WaveCells {
    BinShape shape[64];
    uint32_t start[64];
    uint32_t own[64];
    unsigned long long mask[64];
    uint32_t cnt[64];
};

// Binning with workgroup-local tile histograms in LDS: each workgroup
// projects a.bin_rounds x 256 Gaussians of one frame, counts their
// intersections per tile with LDS atomics (16-bit counts, two tiles per word: a
// count never exceeds BIN_GROUP), stores its histogram and adds it to the frame's tile
// counts with one global atomic per non-empty tile.  The workgroup's pre-sort
// slots are one contiguous range taken with a single atomic and dealt out in
// order of the Gaussians; where the range lies does not matter to any result,
// and no prefix sum over the (frame, Gaussian) counts is needed (960x540 clip
// of 50 frames and 200k Gaussians: prefix sums 73 -> 14 us, this pass 405 -> 425).
// A Gaussian's passing tiles
// are also recorded as a row-major mask over its rectangle (rectangles of at
// most 64 tiles), which the scatter walks.
//
// Work order with dynamics or SH (block_and_frame): B-spline clip 1,050 -> 948
// us, SH clip 937 -> 898 us.  Static scenes (76 bytes) keep the frame-major
// order: 425 us against 448, and 1,349 against 1,564 us at 1080p.
template <bool DYN, bool SH, typename T>
__global__ __launch_bounds__(256) void k_project_lds(Args a) {
    extern __shared__ uint32_t hist[];
    __shared__ WaveCells wc[4];
    constexpr int ROUNDS = BIN_GROUP / 256;  // at most; a small launch takes one
    __shared__ uint16_t counts[ROUNDS][256];  // a Gaussian meets at most LDS_TILE_LIMIT tiles
    __shared__ uint32_t wtotal[ROUNDS][4];
    __shared__ uint32_t slot0;
    static_assert(LDS_TILE_LIMIT <= 0xffff, "16-bit counts");
    int block = blockIdx.x, f = blockIdx.y;
    if ((DYN || SH) && !block_and_frame(a.bin_blocks, a.frames, block, f)) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int words = (a.tiles + 1) >> 1;
    for (int t = threadIdx.x; t < words; t += 256) hist[t] = 0u;
    const CamD cam = uniform_camera(load_camera(a.poses + 7 * f));
    const double tt = a.times ? static_cast<double>(a.times[f]) : static_cast<double>(a.t0);
    __shared__ SplineD basis;
    if (DYN && a.n_ctrl > 0 && threadIdx.x == 0) basis = spline_at(a.n_ctrl, tt);
    __syncthreads();
    const int64_t g0 = static_cast<int64_t>(block) * a.bin_rounds * 256;
    WaveCells& W = wc[w];
#pragma unroll 1
    for (int k = 0; k < a.bin_rounds; ++k) {
        const int64_t g = g0 + k * 256 + threadIdx.x;
        BinShape S;
        const bool has = g < a.n && project_one<DYN, SH, T>(a, f, g, cam, tt, basis, S);
        const uint32_t ncell = has ? static_cast<uint32_t>(S.rw * S.rh) : 0u;
        uint32_t total;
        const uint32_t start = wave_exclusive_scan(ncell, lane, total);
        W.shape[lane] = S;
        W.start[lane] = start;
        W.mask[lane] = 0ull;
        W.cnt[lane] = 0u;
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (uint32_t b0 = 0; b0 < total; b0 += 64) {
            const uint32_t item = b0 + static_cast<uint32_t>(lane);
            const int o = chunk_owner(W.own, start, ncell, b0, lane);
            if (item < total) {
                const uint32_t cell = item - W.start[o];
                const BinShape& So = W.shape[o];
                const int ry = static_cast<int>(cell) / So.rw;
                const int tx = So.tx0 + (static_cast<int>(cell) - ry * So.rw), ty = So.ty0 + ry;
                if (shape_meets_tile(a, So, tx, ty)) {
                    const int tl = ty * a.tiles_x + tx;
                    atomicAdd(&hist[tl >> 1], 1u << ((tl & 1) << 4));
                    atomicAdd(&W.cnt[o], 1u);
                    if (So.rw * So.rh <= 64) atomicOr(&W.mask[o], 1ull << cell);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (g < a.n) {
            const int64_t i = static_cast<int64_t>(f) * a.n + g;
            a.gcnt[i] = W.cnt[lane];
            if (has) a.tmask[i] = W.mask[lane];
        }
        counts[k][threadIdx.x] = static_cast<uint16_t>(W.cnt[lane]);
        __builtin_amdgcn_wave_barrier();
    }
    // the workgroup's slots, in order of the Gaussians
    uint32_t before[ROUNDS] = {};
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        if (k >= a.bin_rounds) break;
        uint32_t total;
        before[k] = wave_exclusive_scan(counts[k][threadIdx.x], lane, total);
        if (lane == 0) wtotal[k][w] = total;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int k = 0; k < a.bin_rounds * 4; ++k) {
            const uint32_t v = wtotal[k >> 2][k & 3];
            wtotal[k >> 2][k & 3] = run;
            run += v;
        }
        slot0 = run ? atomicAdd(&a.status[ST_SLOTS], run) : 0u;
    }
    uint32_t* bh = a.bhist + (static_cast<int64_t>(f) * a.bin_blocks + block) * a.tiles;
    uint32_t* tc = a.tcnt + static_cast<int64_t>(f) * a.tiles;
    for (int t = threadIdx.x; t < a.tiles; t += 256) {
        const uint32_t v = (hist[t >> 1] >> ((t & 1) << 4)) & 0xFFFFu;
        bh[t] = v;
        if (v) atomicAdd(&tc[t], v);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        const int64_t g = g0 + k * 256 + threadIdx.x;
        if (a.goff && k < a.bin_rounds && g < a.n)
            a.goff[static_cast<int64_t>(f) * a.n + g] = slot0 + wtotal[k][w] + before[k];
    }
}

// Write intersection (f, g) -> tile (tx, ty) with pre-sort slot goff + k at
// position next(tile) of the tile's bucket, below end(tile) (the bucket's end
// in the global-atomic scatter; the workspace's capacity in the LDS scatter).
// The counts bound every write; a
// mismatch is an internal error, reported instead of written out of bounds.
template <typename Next, typename End>
__device__ __forceinline__ void emit_key(const Args& a, uint64_t key, uint32_t slot, int tx, int ty, Next next,
                                         End end) {
    const int tl = ty * a.tiles_x + tx;
    const uint32_t pos = next(tl);
    if (pos >= end(tl)) {
        a.status[ST_OVERFLOW] = 2u;
        return;
    }
    KeySlot ks;
    ks.key = key;
    ks.slot = slot;
    ks.pad = 0u;
    a.kv[pos] = ks;
}

// Key (fp32 depth bits << 32 | Gaussian index) of (f, g).
__device__ __forceinline__ uint64_t sort_key(float depth, int64_t g) {
    return (static_cast<uint64_t>(__float_as_uint(depth)) << 32) | static_cast<uint64_t>(g);
}

// Intersections of a Gaussian whose rectangle exceeds 64 tiles (no mask):
// the tests are repeated in the count pass's row-major order.
template <typename Next, typename End>
__device__ __forceinline__ void scatter_big(const Args& a, int64_t g, const Record& r, const BinShape& S,
                                            uint32_t cnt, uint32_t goff, Next next, End end) {
    const uint64_t key = sort_key(r.depth, g);
    uint32_t k = 0;
    for (int ty = S.ty0; ty < S.ty0 + S.rh; ++ty)
        for (int tx = S.tx0; tx < S.tx0 + S.rw; ++tx)
            if (shape_meets_tile(a, S, tx, ty)) {
                if (k >= cnt) {
                    a.status[ST_OVERFLOW] = 2u;
                    return;
                }
                emit_key(a, key, goff + k, tx, ty, next, end);
                ++k;
            }
}

struct WaveKeys {
    unsigned long long mask[64];
    unsigned long long key[64];
    uint32_t start[64];
    uint32_t own[64];
    uint32_t goff[64];
    int tx0[64], ty0[64], rw[64];
};

// Scatter counterpart: one global atomic per non-empty (workgroup, tile)
// reserves the workgroup's range in the tile's bucket; positions inside it are
// handed out by LDS atomics.  A wave deals out its Gaussians' intersections
// (the set bits of their masks) one per lane and step; the k-th set bit of a
// mask gets pre-sort slot goff + k, as the count pass ordered them.
//
// STAGED: written one by one, keys reach memory as 16-byte pieces of lines that
// the L2s cannot hold until their neighbours come (the workgroups in flight
// write some 100 MB): 28 M write requests for the 30 M keys of the 50-frame
// 960x540 clip of 200k Gaussians, most of 32 bytes, and 446 us, with three
// workgroups on a CU as with eight.  So the workgroup collects its keys in LDS
// in order of the tiles, 8 bytes each, and writes a tile's run (three keys
// there) in one go: 335 us; 24 frames of 400k 452 -> 341.  For tile grids of up
// to STAGE_TILES tiles, whose tables leave room for two workgroups of eight
// waves on a CU; a workgroup with more than STAGE_KEYS keys writes them one by
// one.  On few tiles the runs are long enough to fill lines either way, and
// the collecting costs more than it saves: 666 frames of 1,843 Gaussians on 24
// tiles 47 us collected against 37, 250 of 4,915 on 64 tiles 46 against 41, 111
// of 11,059 on 144 tiles 49 against 53 (of smaller Gaussians 37 against 34), 53 of
// 23,040 on 300 tiles 65 against 88.
constexpr int STAGE_TILES_FROM = 128;
constexpr int STAGE_TILES = 2304;
constexpr int STAGE_KEYS = 5120;
constexpr int STAGE_THREADS = 512;
template <bool STAGED>
__global__ __launch_bounds__(STAGED ? STAGE_THREADS : 256) void k_scatter_lds(Args a) {
    if (overflowed(a.status)) return;
    constexpr int NT = STAGED ? STAGE_THREADS : 256;
    // base[t]: next position of this workgroup's range in tile t's bucket; when
    // keys are collected, what to add to a collected key's index to get there
    extern __shared__ uint32_t base[];
    // collected keys (depth bits; bit 30, tile << 16, Gaussian << 6, its
    // intersection), the next index of each tile (16 bits, two tiles per word),
    // and the Gaussians' first slots
    __shared__ uint2 stage[STAGED ? STAGE_KEYS : 1];
    __shared__ uint32_t cursor[STAGED ? STAGE_TILES / 2 : 1];
    __shared__ uint32_t slots[STAGED ? BIN_GROUP : 1];
    __shared__ uint32_t wsum[NT / 64];
    __shared__ WaveKeys wk[NT / 64];
    static_assert(STAGE_TILES <= 1 << 14 && BIN_GROUP <= 1 << 10 && STAGE_KEYS <= 0xffff, "packed");
    const int f = blockIdx.y;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t* bh = a.bhist + (static_cast<int64_t>(f) * a.bin_blocks + blockIdx.x) * a.tiles;
    const int64_t tile0 = static_cast<int64_t>(f) * a.tiles;
    // eight tiles per thread at a time: all counts are requested, then all
    // reservations, so each batch costs two memory round trips, not sixteen
    constexpr int RT = STAGED ? 5 : 8;
    uint32_t mine = 0u;
    for (int t0 = 0; t0 < a.tiles; t0 += NT * RT) {
        uint32_t v[RT], o[RT], lo[RT], hi[RT];
#pragma unroll
        for (int k = 0; k < RT; ++k) {
            const int t = t0 + k * NT + threadIdx.x;
            v[k] = t < a.tiles ? bh[t] : 0u;
        }
#pragma unroll
        for (int k = 0; k < RT; ++k) {
            const int t = t0 + k * NT + threadIdx.x;
            o[k] = lo[k] = hi[k] = 0u;
            if (v[k]) {
                o[k] = atomicAdd(&a.tcur[tile0 + t], v[k]);
                lo[k] = a.toff[tile0 + t];
                hi[k] = a.toff[tile0 + t + 1];
            }
        }
#pragma unroll
        for (int k = 0; k < RT; ++k) {
            const int t = t0 + k * NT + threadIdx.x;
            if (t < a.tiles) {
                const uint32_t b = v[k] ? lo[k] + o[k] : 0u;
                base[t] = b;
                mine += v[k];
                if (v[k] && b + v[k] > hi[k]) a.status[ST_OVERFLOW] = 2u;  // counts disagree: internal error
            }
        }
    }
    bool staged = false;
    uint32_t total_keys = 0u;
    if (STAGED) {
        uint32_t wave_total;
        uint32_t run = wave_exclusive_scan(mine, lane, wave_total);
        if (lane == 0) wsum[w] = wave_total;
        for (int t = threadIdx.x; t < STAGE_TILES / 2; t += NT) cursor[t] = 0u;
        __syncthreads();
        for (int k = 0; k < NT / 64; ++k) {
            run += k < w ? wsum[k] : 0u;
            total_keys += wsum[k];
        }
        staged = total_keys <= STAGE_KEYS;
        if (staged)
            for (int t = threadIdx.x; t < a.tiles; t += NT) {  // this thread's tiles, as above
                const uint32_t v = bh[t];
                if (!v) continue;
                atomicAdd(&cursor[t >> 1], run << ((t & 1) << 4));
                base[t] -= run;
                run += v;
            }
    }
    __syncthreads();
    // next index of a collected key of tile tl
    auto collect = [&](int tl) {
        const uint32_t sh = (tl & 1) << 4;
        return (atomicAdd(&cursor[tl >> 1], 1u << sh) >> sh) & 0xffffu;
    };
    // a workgroup emits exactly its histogram's count per tile; the end
    // checked per key is only the workspace's (no write out of bounds even
    // if the counts disagreed, which the reservation above reports)
    auto next = [&](int tl) {
        if (!staged) return atomicAdd(&base[tl], 1u);
        const uint32_t li = collect(tl);
        if (li < STAGE_KEYS) stage[li].y = 0u;  // written here, not with the others
        return base[tl] + li;
    };
    auto end = [&](int) { return static_cast<uint32_t>(a.k_cap); };
    const int64_t g0 = static_cast<int64_t>(blockIdx.x) * a.bin_rounds * 256;
    const int rounds = STAGED ? BIN_GROUP / NT : a.bin_rounds;
    WaveKeys& W = wk[w];
    // A Gaussian's count, depth, rectangle, mask and slot offset, requested
    // together (one memory round trip; a Gaussian without intersections
    // ignores them), and the next round's requested before this round's keys
    // are dealt out.  Only a Gaussian too large for a mask reads its record.
    struct In {
        uint32_t cnt;
        float depth;
        uint2 rc;
        uint64_t tm;
        uint32_t go;
    };
    auto load_in = [&](int k, In& x) {
        const int64_t g = g0 + k * NT + threadIdx.x;
        const int64_t i = static_cast<int64_t>(f) * a.n + (g < a.n ? g : 0);
        x.cnt = g < a.n ? a.gcnt[i] : 0u;
        x.depth = a.dkey[i];
        x.rc = a.rect[i];
        x.tm = a.tmask[i];
        x.go = a.goff[i];
    };
    In nxt;
    load_in(0, nxt);
    static_assert(BIN_GROUP / 256 <= 32, "one bit per round");
    uint32_t big = 0u;  // rounds whose Gaussian has no mask, scattered after the loop
#pragma unroll 1
    for (int k = 0; k < rounds; ++k) {
        const int64_t g = g0 + k * NT + threadIdx.x;
        const In cur = nxt;
        if (k + 1 < rounds) load_in(k + 1, nxt);
        const uint32_t cnt = cur.cnt;
        const uint2 rc = cur.rc;
        const uint64_t tm = cur.tm;
        const uint32_t go = cur.go;
        const bool small =
            cnt && ((rc.x >> 16) - (rc.x & 0xffff) + 1) * ((rc.y >> 16) - (rc.y & 0xffff) + 1) <= 64u;
        if (staged) slots[k * NT + threadIdx.x] = go;
        uint32_t total;
        const uint32_t first = wave_exclusive_scan(small ? cnt : 0u, lane, total);
        W.start[lane] = first;
        if (small) {
            W.mask[lane] = tm;
            W.key[lane] = sort_key(cur.depth, g);
            W.goff[lane] = go;
            W.tx0[lane] = rc.x & 0xffff;
            W.ty0[lane] = rc.y & 0xffff;
            W.rw[lane] = static_cast<int>(rc.x >> 16) - static_cast<int>(rc.x & 0xffff) + 1;
        }
        __builtin_amdgcn_wave_barrier();
        for (uint32_t b0 = 0; b0 < total; b0 += 64) {
            const uint32_t item = b0 + static_cast<uint32_t>(lane);
            const int o = chunk_owner(W.own, first, small ? cnt : 0u, b0, lane);
            if (item < total) {
                const uint32_t kk = item - W.start[o];
                const uint64_t m = W.mask[o];
                if (kk >= static_cast<uint32_t>(__popcll(m))) {  // counts and mask disagree: internal error
                    a.status[ST_OVERFLOW] = 2u;
                    continue;
                }
                const int bit = kth_set_bit(m, kk);
                const int ry = bit / W.rw[o];
                const int tx = W.tx0[o] + (bit - ry * W.rw[o]), ty = W.ty0[o] + ry;
                if (staged) {
                    const int tl = ty * a.tiles_x + tx;
                    const uint32_t li = collect(tl), gl = static_cast<uint32_t>(k * NT + w * 64 + o);
                    if (li >= STAGE_KEYS) a.status[ST_OVERFLOW] = 2u;  // counts disagree: internal error
                    else stage[li] = make_uint2(static_cast<uint32_t>(W.key[o] >> 32), 1u << 30 | tl << 16 | gl << 6 | kk);
                } else {
                    emit_key(a, W.key[o], W.goff[o] + kk, tx, ty, next, end);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (cnt && !small) big |= 1u << k;
    }
    // Gaussians too large for a mask, out of the pipelined loop, whose registers
    // the rectangle walk would add to: the wave takes them one after the other,
    // 64 cells at a time.  With each lane walking its own Gaussian's rectangle
    // the few largest Gaussians set the time: 960x540 frame of 100k Gaussians
    // 50 us against 21 so, clip of 50 with 200k 475 against 444, 1080p clip of
    // 32 with 500k 1,990 against 1,810.
#pragma unroll 1
    for (int k = 0; k < rounds; ++k) {
        uint64_t m = __ballot((big >> k) & 1u);
        while (m) {
            const int64_t g = g0 + k * NT + w * 64 + __builtin_ctzll(m);
            m &= m - 1;
            const int64_t i = static_cast<int64_t>(f) * a.n + g;
            const Record r = a.rec[i];
            const BinShape S = shape_from_record(r, a.rect[i]);
            const uint64_t key = sort_key(r.depth, g);
            const uint32_t cnt = a.gcnt[i], go = a.goff[i];
            const int cells = S.rw * S.rh;
            uint32_t before = 0;  // passing cells, in the count pass's row-major order
            for (int c0 = 0; c0 < cells; c0 += 64) {
                const int cell = c0 + lane, ry = cell / S.rw;
                const int tx = S.tx0 + (cell - ry * S.rw), ty = S.ty0 + ry;
                const bool meets = cell < cells && shape_meets_tile(a, S, tx, ty);
                const uint64_t pass = __ballot(meets);
                const uint32_t kk = before + static_cast<uint32_t>(__popcll(pass & ((1ull << lane) - 1ull)));
                if (meets) {
                    if (kk >= cnt) a.status[ST_OVERFLOW] = 2u;  // counts disagree: internal error
                    else emit_key(a, key, go + kk, tx, ty, next, end);
                }
                before += static_cast<uint32_t>(__popcll(pass));
            }
        }
    }
    if (!staged) return;
    __syncthreads();
    for (uint32_t li = threadIdx.x; li < total_keys; li += NT) {
        const uint2 e = stage[li];
        if (!(e.y >> 30)) continue;
        const int tl = static_cast<int>(e.y >> 16 & 0x3fffu);
        const uint32_t gl = e.y >> 6 & 0x3ffu, pos = tl < a.tiles ? base[tl] + li : ~0u;
        if (pos >= end(tl)) {
            a.status[ST_OVERFLOW] = 2u;
            continue;
        }
        KeySlot ks;
        ks.key = static_cast<uint64_t>(e.x) << 32 | static_cast<uint64_t>(g0 + gl);
        ks.slot = slots[gl] + (e.y & 63u);
        ks.pad = 0u;
        a.kv[pos] = ks;
    }
}

// Fallback for tile grids too large for an LDS histogram: global atomics per
// intersection, one lane per Gaussian.
template <bool DYN, bool SH, typename T>
__global__ __launch_bounds__(256) void k_project(Args a) {
    const int f = blockIdx.y;
    const int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool live = g < a.n;
    const CamD cam = load_camera(a.poses + 7 * f);
    const double t = a.times ? static_cast<double>(a.times[f]) : static_cast<double>(a.t0);
    SplineD basis = {};
    if (DYN && a.n_ctrl > 0) basis = spline_at(a.n_ctrl, t);
    uint32_t* tc = a.tcnt + static_cast<int64_t>(f) * a.tiles;
    const int64_t i = static_cast<int64_t>(f) * a.n + g;
    BinShape S;
    uint32_t cnt = 0;
    if (live && project_one<DYN, SH, T>(a, f, g, cam, t, basis, S)) {
        uint64_t mask = 0;
        const bool small = S.rw * S.rh <= 64;
        for (int ry = 0; ry < S.rh; ++ry)
            for (int rx = 0; rx < S.rw; ++rx)
                if (shape_meets_tile(a, S, S.tx0 + rx, S.ty0 + ry)) {
                    ++cnt;
                    atomicAdd(&tc[(S.ty0 + ry) * a.tiles_x + S.tx0 + rx], 1u);
                    if (small) mask |= 1ull << (ry * S.rw + rx);
                }
        a.tmask[i] = mask;
    }
    // the wave's slots: one contiguous range
    uint32_t total, slot0 = 0;
    const uint32_t before = wave_exclusive_scan(cnt, lane, total);
    if (lane == 0 && total) slot0 = atomicAdd(&a.status[ST_SLOTS], total);
    slot0 = static_cast<uint32_t>(__shfl(static_cast<int>(slot0), 0, 64));
    if (live) {
        a.gcnt[i] = cnt;
        if (a.goff) a.goff[i] = slot0 + before;
    }
}

__global__ __launch_bounds__(256) void k_scatter(Args a) {
    if (overflowed(a.status)) return;
    const int f = blockIdx.y;
    const int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (g >= a.n) return;
    const int64_t tile0 = static_cast<int64_t>(f) * a.tiles;
    const int64_t i = static_cast<int64_t>(f) * a.n + g;
    const uint32_t cnt = a.gcnt[i];
    if (cnt == 0) return;
    const Record r = a.rec[i];
    const BinShape S = shape_from_record(r, a.rect[i]);
    scatter_big(a, g, r, S, cnt, a.goff[i],
                [&](int tl) { return a.toff[tile0 + tl] + atomicAdd(&a.tcur[tile0 + tl], 1u); },
                [&](int tl) { return a.toff[tile0 + tl + 1]; });
}

// Copy frame 0's projected records out for inspection: (u, v, A00, A01, A11,
// depth, opacity, 0) and the tile count (0 = culled).
__global__ __launch_bounds__(256) void k_export_records(Args a, float* __restrict__ out, int32_t* __restrict__ counts) {
    const int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (g >= a.n) return;
    const uint32_t c = a.gcnt[g];
    counts[g] = static_cast<int32_t>(c);
    float* o = out + 8 * g;
    if (c) {
        const Record r = a.rec[g];
        o[0] = static_cast<float>(r.u);
        o[1] = static_cast<float>(r.v);
        o[2] = r.a;
        o[3] = r.b;
        o[4] = r.c;
        o[5] = r.depth;
        o[6] = a.col4[g].o;  // frame 0
    } else {
        for (int k = 0; k < 7; ++k) o[k] = 0.0f;
    }
    o[7] = 0.0f;
}

hipError_t launch_export_records(const Args& a, float* records, int32_t* counts, hipStream_t stream) {
    if (a.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_export_records, dim3(static_cast<uint32_t>((a.n + 255) / 256)), dim3(256), 0, stream, a,
                       records, counts);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t count, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(static_cast<uint32_t>((count + 255) / 256)), dim3(256), 0, stream, p, value,
                       count);
    return hipGetLastError();
}

int64_t bin_blocks(int64_t n) { return (n + BIN_GROUP - 1) / BIN_GROUP; }

template <bool DYN, bool SH, typename T>
static void launch_projection(const Args& a, hipStream_t stream) {
    const dim3 block(256);
    if (!a.bhist) {
        hipLaunchKernelGGL((k_project<DYN, SH, T>), dim3(static_cast<uint32_t>((a.n + 255) / 256), a.frames), block, 0,
                           stream, a);
        return;
    }
    const size_t lds = sizeof(uint32_t) * ((a.tiles + 1) / 2);
    const uint32_t blocks = static_cast<uint32_t>(a.bin_blocks), frames = static_cast<uint32_t>(a.frames);
    const dim3 grid = DYN || SH ? dim3(XCDS * xcd_share(a.bin_blocks, a.frames)) : dim3(blocks, frames);
    hipLaunchKernelGGL((k_project_lds<DYN, SH, T>), grid, block, lds, stream, a);
}

template <typename T>
static hipError_t launch_project_as(const Args& a, hipStream_t stream) {
    const bool dyn = a.n_ctrl > 0 || a.scale_coeffs || a.quat_coeffs, sh = a.sh_degree > 0;
    const int64_t ft = static_cast<int64_t>(a.frames) * a.tiles, marks = a.pused ? a.k_cap / 32 + 2 : 0;
    const int64_t threads = std::max({static_cast<int64_t>(ST_WORDS), ft, marks, dyn ? int64_t(0) : a.n});
    hipLaunchKernelGGL(k_begin<T>, dim3(static_cast<uint32_t>((threads + 255) / 256)), dim3(256), 0, stream, a, !dyn, ft,
                       marks);
    if (a.n <= 0) return hipGetLastError();
    if (dyn && sh) launch_projection<true, true, T>(a, stream);
    else if (dyn) launch_projection<true, false, T>(a, stream);
    else if (sh) launch_projection<false, true, T>(a, stream);
    else launch_projection<false, false, T>(a, stream);
    return hipGetLastError();
}

// Clears the counters (and the adjoint's marks) and projects; the
// instantiations without dynamics read the shapes the first kernel leaves.
// Without a.goff and a.pused the slots are counted but not handed out.
hipError_t launch_project(const Args& a, hipStream_t stream) {
    return a.dtype == GV_BF16 ? launch_project_as<uint16_t>(a, stream) : launch_project_as<float>(a, stream);
}

hipError_t launch_scatter(const Args& a, hipStream_t stream) {
    if (a.n <= 0) return hipSuccess;
    if (a.bhist) {
        const dim3 grid(static_cast<uint32_t>(a.bin_blocks), a.frames);
        const size_t lds = sizeof(uint32_t) * a.tiles;
        if (a.tiles >= STAGE_TILES_FROM && a.tiles <= STAGE_TILES && a.bin_rounds == BIN_GROUP / 256)
            hipLaunchKernelGGL(k_scatter_lds<true>, grid, dim3(STAGE_THREADS), lds, stream, a);
        else
            hipLaunchKernelGGL(k_scatter_lds<false>, grid, dim3(256), lds, stream, a);
    } else {
        hipLaunchKernelGGL(k_scatter, dim3(static_cast<uint32_t>((a.n + 255) / 256), a.frames), dim3(256), 0, stream,
                           a);
    }
    return hipGetLastError();
}

}  // namespace gv
