// Per-tile depth sort.  The binning pass already grouped the intersections by
// (frame, tile) (a counting sort on the tile digit); each tile's bucket is
// then sorted by the 64-bit key (fp32 depth bits, Gaussian index) by one
// workgroup.  Keys are unique within a bucket, so the order is fully determined
// (depth, ties by lower index) whatever order the atomics of the scatter
// produced and whichever of the ways below sorts it:
//
// * by comparison in one wave (buckets of up to 64 keys);
// * by depth bins in LDS (buckets of up to 2,048 keys at the default setting)
//   or in the merge scratch (longer ones);
// * where more than BIN_KEYS keys fall in one bin (a surface, clusters and
//   outliers), by fine bins, laid out after the keys' distribution;
// * where even those crowd, by merging in a second launch: ranks by comparison
//   within chunks of 16 keys, then by merging pairs of sorted runs level by
//   level (binary search in the other run, the searches of a thread's elements
//   interleaved).  Buckets longer than the LDS capacity are sorted in LDS chunks
//   and merged in global memory (each element finds its place in the partner
//   run by binary search).
//
// Bound by the latency of a bucket's few dependent steps; registers and LDS are
// kept to eight waves per SIMD.  Merging alone took 445 us on the 50-frame
// 960x540 clip of 200k Gaussians, 1,485 us on the 32-frame 1080p clip of 500k
// and 800 us on 24 frames of 400k (buckets beyond 2,048 keys); by bins 295, 960
// and 490 us.  500 frames of 100 Gaussians (four keys to a bucket) 360 us, by bins
// 493, 200 in one wave.  Eight 540p frames of 200k with 80 % of the depths on a wavy
// surface 148 against 106 us, all depths equal 107 against 56.  Two crowds cost
// more than merging alone would: half the depths within 0.001 and half spread 138
// against 214 us, all within 1e-5 (21 values) 137 against 205; the attempt by depth
// bins takes 60 of them, putting the keys in the scratch 70.  (In registers, fine
// bins or bins split where they crowd spill at eight waves per SIMD, which costs
// every bucket 40 % and more; leaving crowds to the merges at once 257.)
#include "gv_internal.h"

#include <algorithm>

namespace gv {

// Keys that pad the LDS buffers: above every real key (whose high word is the
// bit pattern of a finite depth) and distinct from each other.
__device__ __forceinline__ uint64_t pad_key(int e) { return 0xFFFFFFFF00000000ull | static_cast<uint32_t>(e); }

// Adds to rank[j0 + j] (j < NJ) the number of keys below x[j0 + j] in the
// sorted run of R keys at S + st[j0 + j] (R a power of two; slots past the
// run's keys hold keys above every real key): binary lifting, unrolled, the
// NJ searches interleaved so that their LDS reads are in flight together.
template <int R, int NJ, int EPT>
__device__ __forceinline__ void count_below_n(const uint64_t* S, int j0, const int (&st)[EPT],
                                              const uint64_t (&x)[EPT], int (&rank)[EPT]) {
    const uint64_t* p[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) p[j] = S + st[j0 + j];
#pragma unroll
    for (int step = R / 2; step >= 1; step /= 2) {
        uint64_t y[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) y[j] = p[j][step - 1];
#pragma unroll
        for (int j = 0; j < NJ; ++j) p[j] = y[j] < x[j0 + j] ? p[j] + step : p[j];
    }
    uint64_t y[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) y[j] = p[j][0];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        rank[j0 + j] += static_cast<int>(p[j] - (S + st[j0 + j])) + (y[j] < x[j0 + j] ? 1 : 0);
}

// count_below_n over the elements j of this wave that hold a key, j < EPT:
// element j of thread t is e = t + WG j, so they are a prefix of j, the same
// for the whole wave ((t & ~63) + WG j < live).  Up to four searches are
// interleaved at a time.  Lanes whose e is past `live` search as well (every
// window lies inside the buffer) and their results are ignored.
template <int R, int EPT>
__device__ __forceinline__ void count_below_wave(const uint64_t* S, int live, const int (&st)[EPT],
                                                 const uint64_t (&x)[EPT], int (&rank)[EPT]) {
    const int w0 = static_cast<int>(threadIdx.x) & ~63;
#pragma unroll
    for (int j0 = 0; j0 < EPT; j0 += 4) {
        int nj = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) nj += (j0 + j < EPT && w0 + WG * (j0 + j) < live) ? 1 : 0;
        if (nj == 0) break;
        if (nj == 4 && j0 + 4 <= EPT) count_below_n<R, (EPT < 4 ? EPT : 4), EPT>(S, j0, st, x, rank);
        else if (nj >= 3 && EPT >= 3) count_below_n<R, (EPT < 3 ? EPT : 3), EPT>(S, j0, st, x, rank);
        else if (nj >= 2 && EPT >= 2) count_below_n<R, (EPT < 2 ? EPT : 2), EPT>(S, j0, st, x, rank);
        else count_below_n<R, 1, EPT>(S, j0, st, x, rank);
        if (nj < 4) break;
    }
}

// count_below_wave for a run length known only at run time (a power of two,
// R <= runlen <= CAP).
template <int R, int CAP>
__device__ __forceinline__ void count_below_wave_upto(const uint64_t* S, int runlen, int live,
                                                      const int (&st)[CAP / WG], const uint64_t (&x)[CAP / WG],
                                                      int (&rank)[CAP / WG]) {
    if constexpr (R < CAP) {
        if (runlen > R) {
            count_below_wave_upto<2 * R, CAP>(S, runlen, live, st, x, rank);
            return;
        }
    }
    count_below_wave<R, CAP / WG>(S, live, st, x, rank);
}

// Merge levels R, 2R, ... below npad: a key's rank in the merged pair of runs
// is its rank in its own run plus the number of the other run's keys below it.
// Each level reads `cur` and writes its merged runs to `nxt`; the buffers
// swap after every level.
template <int R, int CAP>
__device__ __forceinline__ void merge_levels(uint64_t*& cur, uint64_t*& nxt, int npad, const uint64_t (&x)[CAP / WG],
                                             int (&rank)[CAP / WG]) {
    constexpr int EPT = CAP / WG;
    if constexpr (R < CAP) {
        if (R >= npad) return;
        // the thread index passes through an empty asm statement, so that the
        // compiler cannot compute every level's windows up front (registers)
        int t = static_cast<int>(threadIdx.x);
        asm volatile("" : "+v"(t));
        int st[EPT];
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const int e = t + WG * j;
            const int gb = e & ~(2 * R - 1);  // first element of the pair of runs
            st[j] = (e & R) ? gb : gb + R;    // the other run
        }
        count_below_wave<R, EPT>(cur, npad, st, x, rank);
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const int e = t + WG * j;
            if (e < npad) nxt[(e & ~(2 * R - 1)) + rank[j]] = x[j];
        }
        __syncthreads();
        uint64_t* tmp = cur;
        cur = nxt;
        nxt = tmp;
        merge_levels<2 * R, CAP>(cur, nxt, npad, x, rank);
    }
}

// Ranks of the keys of one bucket segment of len <= CAP keys, in LDS.
// Thread t owns elements e = t + WG j (their keys and values stay in
// registers; only keys are exchanged through LDS).  Level 0 ranks every key
// within its chunk of 16 by comparison with the chunk's keys; each following
// level merges pairs of sorted runs (16 -> 32 -> 64 -> ...).  Each level
// writes its sorted runs (key at its rank) for the next level's searches.
// Padding keys lie above every real key (real depths are finite) and are
// distinct, so the ranks of a level are a permutation and every slot is
// written.  Returns the buffer (SA or SB) holding the keys in sorted order.
template <int CAP>
__device__ __forceinline__ uint64_t* lds_sort_ranks(const KeySlot* src, int len, uint64_t* SA, uint64_t* SB,
                                               uint64_t (&x)[CAP / WG], uint32_t (&v)[CAP / WG],
                                               int (&rank)[CAP / WG]) {
    constexpr int EPT = CAP / WG;
    int t = static_cast<int>(threadIdx.x);  // see merge_levels
    asm volatile("" : "+v"(t));
    const int npad = (len + 15) & ~15;
    // the last level merges groups of `top` keys; slots [npad, top) of both
    // buffers keep padding keys, so every run searched has its full length
    int top = 16;
    while (top < npad) top <<= 1;
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
        const int e = t + WG * j;
        if (e < len) {
            const KeySlot ks = src[e];
            x[j] = ks.key;
            v[j] = ks.slot;
        } else {
            x[j] = pad_key(e);
            v[j] = 0u;
        }
        if (e < npad) SA[e] = x[j];
        else if (e < top) SA[e] = SB[e] = pad_key(e);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
        const int e = t + WG * j;
        rank[j] = 0;
        if (e < npad) {
            const uint64_t* C = SA + (e & ~15);
            int r = 0;
#pragma unroll
            for (int k = 0; k < 16; ++k) r += C[k] < x[j] ? 1 : 0;
            rank[j] = r;
            SB[(e & ~15) + r] = x[j];
        }
    }
    __syncthreads();
    uint64_t* cur = SB;
    uint64_t* nxt = SA;
    merge_levels<16, CAP>(cur, nxt, npad, x, rank);
    return cur;
}

// Number of elements of the sorted run R[0, len) whose key is strictly smaller.
__device__ __forceinline__ int64_t lower_rank(const KeySlot* R, int64_t len, uint64_t key) {
    int64_t lo = 0, hi = len;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (R[mid].key < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// Sorting by depth bins.  The bucket's depths (as bit patterns) are cut into
// bins of one power-of-two width between the smallest and the largest; a key's
// rank is the number of keys in the bins before its own (a prefix sum of LDS
// counts) plus the smaller keys of its own bin, found by comparing with each.
// With at least as many bins as keys that is a handful of LDS accesses per key,
// where merging runs of n keys takes about (log2 n)^2 / 2 dependent ones.

// Inclusive prefix sum over the wave's 64 lanes.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x) {
    x += __builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0u, x, 0x142, 0xa, 0xf, false);  // row_bcast 15, 31
    x += __builtin_amdgcn_update_dpp(0u, x, 0x143, 0xc, 0xf, false);
    return x;
}

// Largest x of the wave, in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false)));
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false)));
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false)));
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false)));
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x142, 0xa, 0xf, false)));
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x143, 0xc, 0xf, false)));
    return __builtin_amdgcn_readlane(x, 63);
}

// Bins (d - lo) >> shift of the keys' upper words d (the depths) or, where
// those are all equal, their lower words (the indices).
struct DepthBins {
    uint32_t lo;
    int shift, word;  // word: 32 or 0
    __device__ __forceinline__ int operator()(uint64_t key) const {
        return static_cast<int>((static_cast<uint32_t>(key >> word) - lo) >> shift);
    }
};

// 2^log_nb bins between the smallest and the largest of the words that for_keys
// passes to its argument.  Uniform over the workgroup; one barrier, two for
// equal depths.  `red` holds four words per wave.
template <typename ForKeys>
__device__ __forceinline__ DepthBins depth_bins(int log_nb, uint32_t* red, const ForKeys& for_keys) {
    const int w = static_cast<int>(threadIdx.x) >> 6;
    DepthBins B;
    for (B.word = 32;; B.word = 0) {
        uint32_t lo = ~0u, hi = 0u;
        for_keys([&](uint64_t x) {
            const uint32_t d = static_cast<uint32_t>(x >> B.word);
            lo = min(lo, d);
            hi = max(hi, d);
        });
        lo = ~wave_max(~lo);
        hi = wave_max(hi);
        if ((threadIdx.x & 63) == 0) {
            red[w] = lo;
            red[WG / 64 + w] = hi;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < WG / 64; ++k) {
            lo = min(lo, red[k]);
            hi = max(hi, red[WG / 64 + k]);
        }
        B.lo = lo;
        const int bits = 32 - __builtin_clz((hi - lo) | 1u);  // hi - lo < 2^bits
        B.shift = bits > log_nb ? bits - log_nb : 0;
        if (hi != lo || B.word == 0) return B;
        red += 2 * (WG / 64);  // the other words may still be read
    }
}

// Counts of K * WG bins to the number of keys in the bins before each.  The
// largest count is returned in every thread; `red` holds two words per wave.
// Contains one barrier; the sums may be read after another.
template <int K>
__device__ __forceinline__ uint32_t scan_bins_of(uint32_t* bins, uint32_t* red) {
    const int t = static_cast<int>(threadIdx.x), w = t >> 6;
    uint32_t c[K], sum = 0u, top = 0u;
#pragma unroll
    for (int k = 0; k < K; ++k) c[k] = bins[t * K + k];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        sum += c[k];
        top = max(top, c[k]);
    }
    const uint32_t incl = wave_inclusive_sum(sum);
    top = wave_max(top);
    if ((t & 63) == 63) {
        red[w] = incl;
        red[WG / 64 + w] = top;
    }
    __syncthreads();
    uint32_t run = incl - sum;
#pragma unroll
    for (int k = 0; k < WG / 64; ++k) {
        run += k < w ? red[k] : 0u;
        top = max(top, red[WG / 64 + k]);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        bins[t * K + k] = run;
        run += c[k];
    }
    return top;
}

__device__ __forceinline__ uint32_t scan_bins(uint32_t* bins, int log_nb, uint32_t* red) {
    static_assert(WG == 256, "one to sixteen bins per thread");
    switch (log_nb) {
        case 8: return scan_bins_of<1>(bins, red);
        case 9: return scan_bins_of<2>(bins, red);
        case 10: return scan_bins_of<4>(bins, red);
        case 11: return scan_bins_of<8>(bins, red);
        default: return scan_bins_of<16>(bins, red);
    }
}

constexpr int64_t MERGE_GROUPS = 1536;  // six per CU, as many as are resident

// Most keys of a bin, each of which is compared with the others.
constexpr uint32_t BIN_KEYS = 64;

// Words of LDS that a sort of buckets of up to CAP keys takes: the bins, and
// then, in their place, the keys.
template <int CAP>
constexpr int SORT_LDS = CAP < 2048 ? 4096 : 2 * CAP;

// Bins for crowded depths (a surface, or clusters and outliers): 256 coarse
// bins by depth, each cut into bins in proportion to its keys between its own
// smallest and largest key.  The keys' whole 64 bits count, so equal depths are
// told apart by their indices.
struct FineBins {
    const uint64_t *lo, *hi;  // [256] keys
    const uint32_t* start;    // [256] keys before
    DepthBins coarse;
    uint32_t n;
    float per_key;  // bins
    int last;       // bin
    // Never falls from a key to a larger one: each float step is monotone.
    __device__ __forceinline__ int operator()(uint64_t x) const {
        const int c = coarse(x);
        const uint32_t s = start[c], cnt = (c < 255 ? start[c + 1] : n) - s;
        const uint64_t l = lo[c], h = hi[c];
        const float f = h > l ? fminf(static_cast<float>(x - l) * (1.0f / static_cast<float>(h - l)), 1.0f) : 0.0f;
        return min(static_cast<int>((static_cast<float>(s) + f * static_cast<float>(cnt)) * per_key), last);
    }
};
constexpr int FINE_WORDS = 5 * 256;  // FineBins' tables

// Fills the coarse tables in `lds` from the keys that for_keys passes to its
// argument and clears the 2^log_nb fine bins.  Ends with a barrier.
template <typename ForKeys>
__device__ __forceinline__ FineBins fine_bins(uint32_t* lds, uint32_t* bins, uint32_t* red, DepthBins coarse, uint32_t n,
                                              int log_nb, const ForKeys& for_keys) {
    static_assert(WG == 256, "a thread per coarse bin");
    const int t = static_cast<int>(threadIdx.x);
    unsigned long long* lo = reinterpret_cast<unsigned long long*>(lds);
    unsigned long long* hi = lo + 256;
    uint32_t* start = lds + 1024;
    __syncthreads();  // the depth bins are no longer read
    lo[t] = ~0ull;
    hi[t] = 0ull;
    start[t] = 0u;
    for (int b = t; b < 1 << log_nb; b += WG) bins[b] = 0u;
    __syncthreads();
    for_keys([&](uint64_t x) {
        const int c = coarse(x);
        if (x < lo[c]) atomicMin(&lo[c], static_cast<unsigned long long>(x));  // (atomics of a crowd wait for each other)
        if (x > hi[c]) atomicMax(&hi[c], static_cast<unsigned long long>(x));
        atomicAdd(&start[c], 1u);
    });
    __syncthreads();
    scan_bins_of<1>(start, red);
    __syncthreads();
    FineBins F;
    F.lo = reinterpret_cast<const uint64_t*>(lo);
    F.hi = reinterpret_cast<const uint64_t*>(hi);
    F.start = start;
    F.coarse = coarse;
    F.n = n;
    F.last = (1 << log_nb) - 1;
    F.per_key = static_cast<float>(1 << log_nb) / static_cast<float>(n);
    return F;
}

// Sort of a bucket of n <= CAP keys by depth bins in LDS; false, with nothing
// written, if the depths crowd in one bin.
template <int CAP>
__device__ __forceinline__ bool bin_sort_lds(const Args& a, uint32_t s, int n, uint32_t* bins, uint32_t* red) {
    constexpr int EPT = CAP / WG;
    constexpr int LOG_MAX = CAP >= 2048 ? 11 : 10;
    static_assert(CAP <= 0xffff, "a bin's start and count share a word");
    const int t = static_cast<int>(threadIdx.x);
    const KeySlot* src = a.kv + s;
    const int log_nb = min(max(33 - __builtin_clz(n), 8), LOG_MAX);  // one to four bins a key, or as many as there are
    uint64_t x[EPT];
    uint32_t v[EPT];
#pragma unroll
    for (int j = 0; j < EPT; ++j)
        if (t + WG * j < n) {
            const KeySlot ks = src[t + WG * j];
            x[j] = ks.key;
            v[j] = ks.slot;
        }
    for (int b = t; b < 1 << log_nb; b += WG) bins[b] = 0u;
    const DepthBins B = depth_bins(log_nb, red, [&](const auto& each) {
#pragma unroll
        for (int j = 0; j < EPT; ++j)
            if (t + WG * j < n) each(x[j]);
    });
    uint32_t at[EPT], fc[EPT];  // place within the bin, then in the bucket; the bin's start and count
#pragma unroll
    for (int j = 0; j < EPT; ++j)
        if (t + WG * j < n) at[j] = atomicAdd(&bins[B(x[j])], 1u);
    __syncthreads();
    if (scan_bins(bins, log_nb, red + 2 * (WG / 64)) > BIN_KEYS) return false;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < EPT; ++j)
        if (t + WG * j < n) {
            const int b = B(x[j]);
            const uint32_t first = bins[b], end = b + 1 < 1 << log_nb ? bins[b + 1] : static_cast<uint32_t>(n);
            at[j] += first;
            fc[j] = first | (end - first) << 16;
        }
    __syncthreads();
    uint64_t* keys = reinterpret_cast<uint64_t*>(bins);
#pragma unroll
    for (int j = 0; j < EPT; ++j)
        if (t + WG * j < n) keys[at[j]] = x[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < EPT; ++j)
        if (t + WG * j < n) {
            const uint32_t first = fc[j] & 0xffffu, end = first + (fc[j] >> 16);
            uint32_t r = first;
            for (uint32_t k = first; k < end; ++k) r += keys[k] < x[j] ? 1u : 0u;
            a.sgid[s + r] = static_cast<uint32_t>(x[j]);
            a.sslot[s + r] = v[j];
        }
    return true;
}

// The same for a longer bucket, or by fine bins: the keys are put in order of
// their bins in the merge scratch, and each is then compared with its bin's keys:
// there, or, for buckets by fine bins of up to FINE_KEYS keys, in LDS (a dozen
// keys to a bin: eight 540p frames with half the depths within 0.001 251 us with
// every comparison a load from the scratch, 224 so).
constexpr int FINE_KEYS = 1536;
template <bool FINE>
__device__ __forceinline__ bool bin_sort_global(const Args& a, uint32_t s, int64_t n, uint32_t* lds, uint32_t* red) {
    constexpr int LOG_NB = 12, LOG_FINE = 11, LOG_LDS = 10;
    static_assert(2 * FINE_KEYS + (1 << LOG_LDS) <= 4096 && FINE_WORDS <= 2 * FINE_KEYS, "keys, and bins behind them");
    if (n > static_cast<int64_t>(BIN_KEYS) << (FINE ? LOG_FINE : LOG_NB)) return false;  // some bin has more
    const int t = static_cast<int>(threadIdx.x);
    const KeySlot* src = a.kv + s;
    KeySlot* dst = a.tkv + s;
    const bool in_lds = FINE && n <= FINE_KEYS;
    auto for_keys = [&](const auto& each) {
        for (int64_t i = t; i < n; i += WG) each(src[i].key);
    };
    auto place = [&](uint32_t* bins, int log_nb, const auto& bin_of) {
        for (int64_t i = t; i < n; i += WG) atomicAdd(&bins[bin_of(src[i].key)], 1u);
        __syncthreads();
        if (scan_bins(bins, log_nb, red + 2 * (WG / 64)) > BIN_KEYS) return false;
        __syncthreads();
        for (int64_t i = t; i < n; i += WG) {
            KeySlot e = src[i];
            e.pad = static_cast<uint32_t>(bin_of(e.key));
            dst[atomicAdd(&bins[e.pad], 1u)] = e;
        }
        __syncthreads();  // bins[b] is now the end of bin b
        uint64_t* keys = reinterpret_cast<uint64_t*>(lds);
        if (in_lds) {
            for (int i = t; i < static_cast<int>(n); i += WG) keys[i] = dst[i].key;
            __syncthreads();
        }
        for (int64_t i = t; i < n; i += WG) {
            const KeySlot e = dst[i];
            const uint32_t first = e.pad ? bins[e.pad - 1] : 0u, end = bins[e.pad];
            uint32_t r = first;
            if (in_lds)
                for (uint32_t k = first; k < end; ++k) r += keys[k] < e.key ? 1u : 0u;
            else
                for (uint32_t k = first; k < end; ++k) r += dst[k].key < e.key ? 1u : 0u;
            a.sgid[s + r] = static_cast<uint32_t>(e.key);
            a.sslot[s + r] = e.slot;
        }
        return true;
    };
    if (FINE) {
        const DepthBins B = depth_bins(8, red, for_keys);
        const int log_nb = in_lds ? LOG_LDS : LOG_FINE;
        uint32_t* bins = lds + (in_lds ? 2 * FINE_KEYS : FINE_WORDS);
        return place(bins, log_nb, fine_bins(lds, bins, red, B, static_cast<uint32_t>(n), log_nb, for_keys));
    }
    for (int b = t; b < 1 << LOG_NB; b += WG) lds[b] = 0u;
    return place(lds, LOG_NB, depth_bins(LOG_NB, red, for_keys));
}

// A bucket of at most a wave's lanes: each lane counts the smaller keys.
__device__ __forceinline__ void wave_sort(const Args& a, uint32_t s, int n) {
    const int lane = static_cast<int>(threadIdx.x);
    KeySlot e = {};
    if (lane < n) e = a.kv[s + lane];
    const uint32_t lo = static_cast<uint32_t>(e.key), hi = static_cast<uint32_t>(e.key >> 32);
    uint32_t r = 0u;
    for (int k = 0; k < n; ++k) {
        const uint64_t x = static_cast<uint64_t>(__builtin_amdgcn_readlane(hi, k)) << 32 | __builtin_amdgcn_readlane(lo, k);
        r += x < e.key ? 1u : 0u;
    }
    if (lane < n) {
        a.sgid[s + r] = lo;
        a.sslot[s + r] = e.slot;
    }
}

// One workgroup per bucket.  A bucket whose keys crowd even in one of the fine
// bins goes on the list of k_tile_merge (in the scatter's cursors, which are no longer needed).
template <int CAP>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(CAP <= 2048 ? 8 : 1))) void k_tile_sort(Args a) {
    if (overflowed(a.status)) return;
    const uint32_t seg = blockIdx.x;
    uint32_t s, e;
    bucket_range(a, seg, s, e);
    if (e <= s) return;
    const uint32_t n = e - s;
    if (n <= 64u) {
        if (threadIdx.x < 64) wave_sort(a, s, static_cast<int>(n));
        return;
    }
    __shared__ __align__(16) uint32_t lds[SORT_LDS<CAP>];
    __shared__ uint32_t red[4 * (WG / 64)];
    if (n <= CAP ? bin_sort_lds<CAP>(a, s, static_cast<int>(n), lds, red) : bin_sort_global<false>(a, s, n, lds, red))
        return;
    __syncthreads();
    if (!bin_sort_global<true>(a, s, n, lds, red) && threadIdx.x == 0) a.tcur[atomicAdd(&a.status[ST_CROWDED], 1u)] = seg;
}

// Sort of one bucket by merging.
template <int CAP>
__device__ __forceinline__ void merge_sort(const Args& a, uint32_t s, int64_t n, uint64_t* SA, uint64_t* SB) {
    constexpr int EPT = CAP / WG;
    uint64_t x[EPT];
    uint32_t v[EPT];
    int rank[EPT];
    KeySlot* src = a.kv + s;
    if (n <= 2 * CAP) {
        // One run, or two: the first is sorted and written back in place, the
        // second sorted in LDS; the first's keys are then reloaded into the
        // other LDS buffer and every element adds the number of keys below it
        // in the other run (binary search in LDS).  One copy of the LDS sort
        // serves both runs.
        const int runs = n <= CAP ? 1 : 2;
        const uint64_t* K1 = nullptr;
#pragma unroll 1
        for (int run = 0; run < runs; ++run) {
            const int len = run == 0 ? (n < CAP ? static_cast<int>(n) : CAP) : static_cast<int>(n) - CAP;
            K1 = lds_sort_ranks<CAP>(src + run * CAP, len, SA, SB, x, v, rank);
            if (run + 1 < runs) {
#pragma unroll
                for (int j = 0; j < EPT; ++j) src[rank[j]] = KeySlot{x[j], v[j], 0u};
                __syncthreads();
            }
        }
        if (runs == 1) {
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                const int i = threadIdx.x + WG * j;
                if (i < n) {
                    a.sgid[s + rank[j]] = static_cast<uint32_t>(x[j]);
                    a.sslot[s + rank[j]] = v[j];
                }
            }
            return;
        }
        const int len1 = static_cast<int>(n) - CAP;
        uint64_t* K0 = K1 == SA ? SB : SA;
        // run 1's keys and padding fill K1[0, top1) (the group size of its last level)
        int top1 = 16;
        while (top1 < ((len1 + 15) & ~15)) top1 <<= 1;
        for (int i = threadIdx.x; i < CAP; i += WG) K0[i] = src[i].key;
        __syncthreads();
        int st[EPT];
#pragma unroll
        for (int j = 0; j < EPT; ++j) st[j] = 0;
        // run 1's elements: their rank in run 1 plus run 0's keys below them
        count_below_wave<CAP, EPT>(K0, len1, st, x, rank);
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const int i = threadIdx.x + WG * j;
            if (i < len1) {
                a.sgid[s + rank[j]] = static_cast<uint32_t>(x[j]);
                a.sslot[s + rank[j]] = v[j];
            }
        }
        // run 0's elements: their position in run 0 plus run 1's keys below them
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const int i = threadIdx.x + WG * j;
            const KeySlot e0 = src[i];
            x[j] = e0.key;
            v[j] = e0.slot;
            rank[j] = i;
        }
        count_below_wave_upto<16, CAP>(K1, top1, CAP, st, x, rank);
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            a.sgid[s + rank[j]] = static_cast<uint32_t>(x[j]);
            a.sslot[s + rank[j]] = v[j];
        }
        return;
    }
    // Long bucket: sorted runs of CAP in place, then pairwise merges.
    KeySlot* dst = a.tkv + s;
    for (int64_t c0 = 0; c0 < n; c0 += CAP) {
        const int len = static_cast<int>(n - c0 < CAP ? n - c0 : CAP);
        // every thread reads its elements of the chunk before the first
        // barrier inside lds_sort_ranks, so the chunk may then be overwritten
        lds_sort_ranks<CAP>(src + c0, len, SA, SB, x, v, rank);
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const int i = threadIdx.x + WG * j;
            if (i < len) src[c0 + rank[j]] = KeySlot{x[j], v[j], 0u};
        }
        __syncthreads();
    }
    for (int64_t w = CAP; w < n; w <<= 1) {
        for (int64_t lo = 0; lo < n; lo += 2 * w) {
            const int64_t mid = lo + w < n ? lo + w : n;
            const int64_t hi = lo + 2 * w < n ? lo + 2 * w : n;
            for (int64_t i = lo + threadIdx.x; i < hi; i += WG) {
                const KeySlot e = src[i];
                int64_t pos;
                if (i < mid) pos = lo + (i - lo) + lower_rank(src + mid, hi - mid, e.key);
                else pos = lo + (i - mid) + lower_rank(src + lo, mid - lo, e.key);
                dst[pos] = e;
            }
        }
        __syncthreads();
        KeySlot* t = src;
        src = dst;
        dst = t;
    }
    for (int64_t i = threadIdx.x; i < n; i += WG) {
        const KeySlot e = src[i];
        a.sgid[s + i] = static_cast<uint32_t>(e.key);
        a.sslot[s + i] = e.slot;
    }
}

// The buckets that k_tile_sort listed, in turn.
template <int CAP>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(CAP <= 1024 ? 6 : 1))) void k_tile_merge(Args a) {
    if (overflowed(a.status)) return;
    __shared__ uint64_t SA[CAP], SB[CAP];
    const uint32_t listed = a.status[ST_CROWDED];
#pragma unroll 1
    for (uint32_t i = blockIdx.x; i < listed; i += gridDim.x) {
        uint32_t s, e;
        bucket_range(a, a.tcur[i], s, e);
        merge_sort<CAP>(a, s, static_cast<int64_t>(e) - s, SA, SB);
        __syncthreads();
    }
}

template <int CAP>
static void launch_sort(const Args& a, int64_t segments, hipStream_t stream) {
    // buckets of up to twice the merges' run length are sorted in LDS
    hipLaunchKernelGGL(k_tile_sort<(CAP < 2048 ? 2 * CAP : 4096)>, dim3(static_cast<uint32_t>(segments)), dim3(WG), 0,
                       stream, a);
    hipLaunchKernelGGL(k_tile_merge<CAP>, dim3(static_cast<uint32_t>(std::min<int64_t>(segments, MERGE_GROUPS))),
                       dim3(WG), 0, stream, a);
}

hipError_t launch_tile_sort(const Args& a, int64_t segments, hipStream_t stream) {
    if (segments <= 0) return hipSuccess;
    switch (a.tune.sort_cap) {
        case 512: launch_sort<512>(a, segments, stream); break;
        case 1024: launch_sort<1024>(a, segments, stream); break;
        case 2048: launch_sort<2048>(a, segments, stream); break;
        default: launch_sort<4096>(a, segments, stream); break;
    }
    return hipGetLastError();
}

}  // namespace gv
