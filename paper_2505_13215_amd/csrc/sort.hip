// Binning and ordering on gfx950 (Alg. 1: DuplicateWithKeys, SortByKeys,
// IdentifyTileRanges).
//
// Design: the per-view depth order is established once over the N Gaussians (by
// float32 depth bits, equal depths by ascending id): by counting, by bins of
// sampled keys, or by a stable LSD radix sort, by length.  Binning is then two-level: every depth-ordered Gaussian emits
// one coarse entry per super-tile (S x S tiles) its square touches, keyed by
// the super-tile and carrying the mask of the super-tile's tiles it reaches.
// Each entry goes straight to its place in its super-tile's depth-ordered list,
// found from per-block histograms and bit masks (ranked binning, k_bin_*); views
// of more super-tiles than a block's masks hold emit their entries and sort
// them stably by super-tile (k_coarse_*).  A tile's list is the sub-sequence of its super-tile's
// list whose mask holds the tile, which the blending kernels compact on the fly
// (64-lane ballot + prefix, walk.hpp): exactly the tile's (depth bits,
// id)-ordered set of overlapping splats - the order a global (tile, depth, id)
// sort gives - without sorting or storing (Gaussian, tile) pairs at all.
//
// When a batched call repeats a camera at several times, the 3D Gaussians are
// sorted and binned once per camera (a static group) onto a super-tile grid of
// the group's own, and each view bins only its 4D Gaussians; the blending
// kernels merge the two lists by depth.
//
// Every LSD pass is: per-block digit histogram -> per-digit scan across blocks
// -> stable scatter.  The stable scatter ranks keys inside a wave with ballots
// (64-lane match on the digit bits), orders the block's tile in LDS and writes
// coalesced runs per digit.
#include "common.hpp"
#include "cull.hpp"
#include "launch.hpp"

namespace h4d {

__device__ __forceinline__ uint64_t read_count(const unsigned long long* dc, uint64_t hc) {
    return dc ? (uint64_t)(*dc) : hc;
}

__device__ __forceinline__ unsigned long long lanemask_lt() {
    const int lane = __lane_id();
    return lane == 0 ? 0ull : ((~0ull) >> (64 - lane));
}

// inclusive-to-exclusive block scan of one value per thread (256 threads)
template <typename T>
__device__ inline T block_exclusive_scan_256(T v, T* s_buf, T& total) {
    // wave scans, then the four wave totals (s_buf[0..3])
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    T incl = v;
    for (int off = 1; off < 64; off <<= 1) {
        const T y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) s_buf[w] = incl;
    __syncthreads();
    T base = (T)0;
    for (int k = 0; k < w; ++k) base += s_buf[k];
    total = s_buf[0] + s_buf[1] + s_buf[2] + s_buf[3];
    __syncthreads();  // s_buf is free again for the caller
    return base + incl - v;
}

// ---------------------------------------------------------------------------
// Radix sort pass (up to 11 bits per pass)
// ---------------------------------------------------------------------------
// In-place exclusive scan of s[0 .. radix) (radix <= 2^MB) by the block's 256
// threads, each owning 2^MB / 256 consecutive digits; returns the total.
template <int MB>
__device__ inline uint32_t block_scan_digits(uint32_t* s, int radix, uint32_t* s_buf) {
    constexpr int DPT = (1 << MB) / kSortThreads;
    const int d0 = threadIdx.x * DPT;
    uint32_t v[DPT];
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < DPT; ++q) {
        v[q] = d0 + q < radix ? s[d0 + q] : 0u;
        sum += v[q];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan_256<uint32_t>(sum, s_buf, total);
#pragma unroll
    for (int q = 0; q < DPT; ++q) {
        if (d0 + q < radix) s[d0 + q] = run;
        run += v[q];
    }
    __syncthreads();
    return total;
}

// MB: largest digit width the instantiation handles (LDS is sized for it).
// skip_empty: keys whose upper 16 bits are zero (coarse entries with an empty
// tile mask) are left out of the counts (and, in the downsweep, of the output).
template <int MB>
__global__ void __launch_bounds__(kSortThreads) k_radix_upsweep(const uint32_t* __restrict__ keys,
                                                                const unsigned long long* dcount, uint64_t hcount,
                                                                int shift, int nbits, uint32_t* __restrict__ hist,
                                                                int nblocks, uint64_t seg_stride, int skip_empty) {
    __shared__ uint32_t s_hist[4][1 << MB];
    const int radix = 1 << nbits;
    keys += (size_t)blockIdx.y * seg_stride;
    hist += (size_t)blockIdx.y * radix * nblocks;
    const uint32_t mask = (uint32_t)radix - 1u;
    const int tid = threadIdx.x, w = tid >> 6;
    const uint64_t n = read_count(dcount, hcount);
    const uint64_t begin = (uint64_t)blockIdx.x * kSortTile;
    if (begin >= n) return;  // blocks past the live count are never scanned (uniform)
    for (int d = tid; d < 4 * radix; d += kSortThreads) s_hist[d / radix][d % radix] = 0;
    __syncthreads();
    for (int k = 0; k < kSortItems; ++k) {
        const uint64_t idx = begin + (uint64_t)k * kSortThreads + tid;
        if (idx < n) {
            const uint32_t key = keys[idx];
            if (!skip_empty || (key >> 16) != 0u) atomicAdd(&s_hist[w][(key >> shift) & mask], 1u);
        }
    }
    __syncthreads();
    for (int d = tid; d < radix; d += kSortThreads)
        hist[(size_t)d * nblocks + blockIdx.x] = s_hist[0][d] + s_hist[1][d] + s_hist[2][d] + s_hist[3][d];
}

// one block per (digit, segment): exclusive scan of that digit's per-block
// counts over the blocks that hold live keys (4 counts per thread per round)
__global__ void __launch_bounds__(256) k_radix_digit_scan(uint32_t* __restrict__ hist, int nblocks, int radix,
                                                          uint32_t* __restrict__ totals,
                                                          const unsigned long long* dcount, uint64_t hcount,
                                                          int tile) {
    __shared__ uint32_t s_buf[256];
    const uint64_t n = read_count(dcount, hcount);
    const int live = (int)min((uint64_t)nblocks, (n + tile - 1) / tile);
    uint32_t* h = hist + (size_t)blockIdx.y * radix * nblocks + (size_t)blockIdx.x * nblocks;
    totals += (size_t)blockIdx.y * radix;
    uint32_t carry = 0;
    for (int start = 0; start < live; start += 1024) {
        const int i0 = start + 4 * (int)threadIdx.x;
        uint32_t v[4];
        uint32_t sum = 0;
        for (int q = 0; q < 4; ++q) {
            v[q] = i0 + q < live ? h[i0 + q] : 0u;
            sum += v[q];
        }
        uint32_t tot;
        uint32_t ex = block_exclusive_scan_256<uint32_t>(sum, s_buf, tot) + carry;
        for (int q = 0; q < 4; ++q) {
            if (i0 + q < live) h[i0 + q] = ex;
            ex += v[q];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

template <int MB>
__global__ void __launch_bounds__(kSortThreads) k_radix_downsweep(
    const uint32_t* __restrict__ keys_in, const uint32_t* __restrict__ vals_in, uint32_t* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, const unsigned long long* dcount, uint64_t hcount, int shift, int nbits,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ totals, int nblocks,
    const unsigned long long* out_offset, uint64_t seg_stride, int64_t* __restrict__ digit_ranges, int n_digit_ranges,
    const uint32_t* __restrict__ val_map, int skip_empty, unsigned long long* out_count,
    uint2* __restrict__ pairs_out, uint32_t val0) {
    __shared__ uint32_t s_wcount[4][1 << MB];
    __shared__ uint32_t s_dstart[1 << MB];
    __shared__ uint32_t s_gbase[1 << MB];
    __shared__ uint32_t s_buf[256];
    constexpr int ITEMS = kSortItems, TILE = kSortTile;
    __shared__ uint32_t s_keys[TILE];
    __shared__ uint32_t s_vals[TILE];

    const uint64_t n = read_count(dcount, hcount);
    const uint64_t begin = (uint64_t)blockIdx.x * TILE;
    if (begin >= n) {  // uniform over the block
        // no keys at all: the kept count is still written (block 0 holds keys otherwise)
        if (out_count && n == 0 && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *out_count = 0ull;
        return;
    }
    const int radix = 1 << nbits;
    {
        const size_t so = (size_t)blockIdx.y * seg_stride;
        keys_in += so; keys_out += so; vals_out += so;
        if (vals_in) vals_in += so;
        hist += (size_t)blockIdx.y * radix * nblocks;
        totals += (size_t)blockIdx.y * radix;
    }
    const uint32_t mask = (uint32_t)radix - 1u;
    const int tid = threadIdx.x, w = tid >> 6, lane = __lane_id();

    for (int d = tid; d < 4 * radix; d += kSortThreads) s_wcount[d / radix][d % radix] = 0;
    // global base of digit d = (exclusive scan of totals)[d] + this block's scanned count
    for (int d = tid; d < radix; d += kSortThreads) s_gbase[d] = totals[d];
    __syncthreads();
    const uint32_t n_out = block_scan_digits<MB>(s_gbase, radix, s_buf);
    if (out_count && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *out_count = n_out;
    const unsigned long long off = out_offset ? *out_offset : 0ull;
    // a single-pass sort over whole keys: the digit runs are the key ranges
    if (digit_ranges && blockIdx.x == 0 && blockIdx.y == 0)
        for (int d = tid; d < n_digit_ranges; d += kSortThreads) {
            digit_ranges[2 * (size_t)d] = (int64_t)off + s_gbase[d];
            digit_ranges[2 * (size_t)d + 1] = (int64_t)off + s_gbase[d] + totals[d];
        }
    for (int d = tid; d < radix; d += kSortThreads) s_gbase[d] += hist[(size_t)d * nblocks + blockIdx.x];

    // wave w owns items [begin + w * 64 ITEMS, begin + (w + 1) * 64 ITEMS), ITEMS rounds of 64
    uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
    const unsigned long long lt = lanemask_lt();
    for (int r = 0; r < ITEMS; ++r) {
        const uint64_t idx = begin + (uint64_t)w * (ITEMS * 64) + (uint64_t)r * 64 + lane;
        key[r] = idx < n ? keys_in[idx] : 0u;
        const bool valid = idx < n && (!skip_empty || (key[r] >> 16) != 0u);
        val[r] = !valid ? 0u : vals_in ? vals_in[idx] : val0 + (uint32_t)idx;
        const uint32_t d = (key[r] >> shift) & mask;
        unsigned long long peers = __ballot(valid);
        for (int b = 0; b < nbits; ++b) {
            const bool bit = (d >> b) & 1u;
            const unsigned long long m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t before = (uint32_t)__popcll(peers & lt);
        uint32_t base = 0;
        if (valid) base = s_wcount[w][d];
        rank[r] = base + before;
        if (valid && before == 0) s_wcount[w][d] = base + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    // per digit: prefix over waves, block total per digit, then start of each
    // digit's run in the block-sorted tile
    for (int d = tid; d < radix; d += kSortThreads) {
        uint32_t run = 0;
        for (int q = 0; q < 4; ++q) {
            const uint32_t c = s_wcount[q][d];
            s_wcount[q][d] = run;
            run += c;
        }
        s_dstart[d] = run;
    }
    __syncthreads();
    const int cnt = (int)block_scan_digits<MB>(s_dstart, radix, s_buf);  // keys this block places
    for (int r = 0; r < ITEMS; ++r) {
        const uint64_t idx = begin + (uint64_t)w * (ITEMS * 64) + (uint64_t)r * 64 + lane;
        if (idx < n && (!skip_empty || (key[r] >> 16) != 0u)) {
            const uint32_t d = (key[r] >> shift) & mask;
            const uint32_t pos = s_dstart[d] + s_wcount[w][d] + rank[r];
            s_keys[pos] = key[r];
            s_vals[pos] = val[r];
        }
    }
    __syncthreads();
    for (int p = tid; p < cnt; p += kSortThreads) {
        const uint32_t k = s_keys[p];
        const uint32_t d = (k >> shift) & mask;
        const uint64_t dst = off + (uint64_t)s_gbase[d] + (uint64_t)(p - (int)s_dstart[d]);
        const uint32_t v = val_map ? val_map[s_vals[p]] : s_vals[p];
        if (pairs_out) {
            pairs_out[dst] = make_uint2(k, v);
        } else {
            keys_out[dst] = k;
            vals_out[dst] = v;
        }
    }
}

int radix_blocks(uint64_t capacity, int items) {
    const uint64_t tile = (uint64_t)kSortThreads * items;
    return (int)((capacity + tile - 1) / tile);
}
size_t radix_hist_words(uint64_t capacity, int n_seg, int max_bits, int items) {
    return ((size_t)1 << max_bits) * (size_t)std::max(1, radix_blocks(capacity, items)) * (size_t)std::max(1, n_seg);
}

bool radix_pass_fits(uint64_t capacity, int n_seg, int nbits, int items, size_t hist_words, size_t totals_words) {
    if (nbits < 1 || nbits > kMaxRadixBits || n_seg < 0 || (items != 2 && items != kSortItems)) return false;
    if (items == 2 && nbits > 8) return false;
    return radix_hist_words(capacity, n_seg, nbits, items) <= hist_words &&
           ((size_t)1 << nbits) * (size_t)std::max(1, n_seg) <= totals_words;
}

bool launch_radix_pass(const uint32_t* keys_in, const uint32_t* vals_in, uint32_t* keys_out, uint32_t* vals_out,
                       const unsigned long long* dcount, uint64_t hcount, uint64_t capacity, int shift, int nbits,
                       uint32_t* hist, size_t hist_words, uint32_t* totals, size_t totals_words,
                       const unsigned long long* out_offset, hipStream_t st, int n_seg, uint64_t seg_stride,
                       int64_t* digit_ranges, int n_digit_ranges, const uint32_t* val_map, int skip_empty,
                       unsigned long long* out_count, uint2* pairs_out, uint32_t val0) {
    // every block writes 2^nbits counts per segment: refuse a pass whose
    // histogram or digit totals would not fit the buffers it was given
    if (!radix_pass_fits(capacity, n_seg, nbits, kSortItems, hist_words, totals_words)) return false;
    const int nb = radix_blocks(capacity, kSortItems);
    if (nb == 0 || n_seg == 0) return true;
    const dim3 grid(nb, n_seg);
    // the smallest instantiation that holds the digit (LDS is sized by it)
#define H4D_RADIX_PASS(MB)                                                                                            \
    do {                                                                                                              \
        k_radix_upsweep<MB><<<grid, kSortThreads, 0, st>>>(keys_in, dcount, hcount, shift, nbits, hist, nb,           \
                                                          seg_stride, skip_empty);                                   \
        k_radix_digit_scan<<<dim3(1 << nbits, n_seg), 256, 0, st>>>(hist, nb, 1 << nbits, totals, dcount, hcount,     \
                                                                    kSortTile);                                      \
        k_radix_downsweep<MB><<<grid, kSortThreads, 0, st>>>(                                                        \
            keys_in, vals_in, keys_out, vals_out, dcount, hcount, shift, nbits, hist, totals, nb, out_offset,         \
            seg_stride, digit_ranges, n_digit_ranges, val_map, skip_empty, out_count, pairs_out, val0);               \
    } while (0)
    if (nbits <= 8) H4D_RADIX_PASS(8);
    else if (nbits == 9) H4D_RADIX_PASS(9);
    else if (nbits == 10) H4D_RADIX_PASS(10);
    else H4D_RADIX_PASS(kMaxRadixBits);
#undef H4D_RADIX_PASS
    return true;
}

// ---------------------------------------------------------------------------
// Short sorts: ranks by counting, in one launch.
// ---------------------------------------------------------------------------
// A key's place is the number of keys before it: smaller ones, and equal ones
// of a smaller index (stable).  A workgroup places 64 keys, one per lane; its
// sixteen waves each count over a sixteenth of the segment, whose keys are
// wave-uniform (scalar loads), two instructions per pair.  Bound by instruction
// issue at n^2 / 32 wave instructions, against twelve launches of the radix sort,
// each nearly empty: 2,000 keys 0.045 -> 0.005 ms, 16,000 0.049 -> 0.026 ms.
constexpr int kRankWaves = 16;
// Keys of [j0, j1) that lie before key (EQUAL: or equal it), sixteen scalar
// loads ahead of their comparisons.
template <bool EQUAL>
__device__ __forceinline__ uint32_t rank_count(const uint32_t* __restrict__ keys, int j0, int j1, uint32_t key) {
    constexpr int U = 16;
    uint32_t r = 0u;
    int j = j0;
    if (j + U <= j1) {
        uint32_t k[U];
#pragma unroll
        for (int q = 0; q < U; ++q) k[q] = keys[j + q];
        for (; j + 2 * U <= j1; j += U) {
            uint32_t next[U];
#pragma unroll
            for (int q = 0; q < U; ++q) next[q] = keys[j + U + q];
#pragma unroll
            for (int q = 0; q < U; ++q) r += (EQUAL ? k[q] <= key : k[q] < key) ? 1u : 0u;
#pragma unroll
            for (int q = 0; q < U; ++q) k[q] = next[q];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) r += (EQUAL ? k[q] <= key : k[q] < key) ? 1u : 0u;
        j += U;
    }
    for (; j < j1; ++j) r += (EQUAL ? keys[j] <= key : keys[j] < key) ? 1u : 0u;
    return r;
}

__global__ void __launch_bounds__(64 * kRankWaves) k_rank_sort(const uint32_t* __restrict__ keys,
                                                             uint32_t val0, uint32_t* __restrict__ vals_out,
                                                             int n) {
    __shared__ uint32_t s_rank[kRankWaves][64];
    const size_t seg = (size_t)blockIdx.y * n;
    keys += seg;
    vals_out += seg;
    const int lane = __lane_id(), w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i0 = (int)blockIdx.x * 64, i = i0 + lane;
    const uint32_t key = i < n ? keys[i] : 0u;
    // the wave's keys [j0, j1); those before i0 count when equal too, those from
    // i0 + 64 on only when smaller, and the block's own by index
    const int per = (n + kRankWaves - 1) / kRankWaves;
    const int j0 = min(n, w * per), j1 = min(n, j0 + per);
    uint32_t r = rank_count<true>(keys, j0, min(j1, i0), key);
    for (int j = max(j0, i0); j < min(j1, i0 + 64); ++j) {
        const uint32_t k = keys[j];
        r += (k < key || (k == key && j < i)) ? 1u : 0u;
    }
    r += rank_count<false>(keys, max(j0, i0 + 64), j1, key);
    s_rank[w][lane] = r;
    __syncthreads();
    if (w == 0 && i < n) {
        uint32_t at = 0u;
#pragma unroll
        for (int q = 0; q < kRankWaves; ++q) at += s_rank[q][lane];
        vals_out[at] = val0 + (uint32_t)i;
    }
}

// ---------------------------------------------------------------------------
// Longer depth sorts: bins between sampled keys, each bin ordered in LDS.
// ---------------------------------------------------------------------------
// Keys are ordered as 64-bit pairs (depth bits, id), which are all different, so
// bins of a fixed share of the keys exist for any input (equal depths and culled
// splats included), a bin's keys may arrive in any order, and the result is the
// stable order.  Four samples per bin, one at a hashed place of each equal stretch
// of the segment, give the bounds; a counting and a scattering launch move the keys
// to their bins, and one workgroup per bin orders it.  The keys are read twice and
// moved once (an 8-bit radix sort reads them eight times and moves them four), in
// four or five launches instead of twelve: 18,000 keys 0.054 -> 0.023 ms, 250,000
// 0.065 -> 0.040, 500,000 0.079 -> 0.052, eight segments of 500,000 0.212 -> 0.150.
// Short segments are bound by the launches and one trip through memory in each,
// long ones by the searches in LDS (k_depth_bins, 19 ns per 1000 keys).
constexpr int kSplitThreads = 1024;
constexpr int kSplitOver = 4;
constexpr int kSplitMaxBins = 2048;
// Up to here a scatter workgroup sums the counting workgroups' rows itself, a load
// per row; beyond, a launch scans them first.
constexpr int kSplitDirect = 64;
// From this many samples on a launch gathers them once: one segment of 1M (8192
// samples) 0.087 -> 0.075 ms, eight of 500,000 0.176 -> 0.150; 250,000 (4096) even.
constexpr size_t kSplitGather = 8192;
constexpr int kBinWaves = 8;
constexpr int kBinKeys = 4096;  // a bin's keys held in LDS (32 KB)

// The radix sort takes the longest segments, whose bins and runs grow: 1M keys 0.075
// ms here against 0.100, four segments of 1M 0.169 against 0.208, 2M 0.154 against
// 0.125.
DepthPlan depth_plan(int n, int n_seg) {
    DepthPlan p;
    const bool large = n > (1 << 19);
    p.radix = n > (1 << 20);
    p.lg_bins = 6;
    while (p.lg_bins < (large ? 11 : 10) && ((int64_t)256 << p.lg_bins) < n) ++p.lg_bins;
    p.items = large ? 8 : 4;
    p.blocks = (int)(((int64_t)n + kSplitThreads * p.items - 1) / (kSplitThreads * p.items));
    // per segment and bin: the bound (64 bits), total, start, four samples, and a row
    // per workgroup
    p.words = p.radix ? radix_hist_words((uint64_t)n, n_seg, kDepthDigitBits, kSortItems)
                      : ((size_t)n_seg << p.lg_bins) * (4 + kSplitOver + (size_t)p.blocks);
    return p;
}

// Place of sample j of 2^lg: a hashed one of [j n / 2^lg, (j + 1) n / 2^lg).
__device__ __forceinline__ int sample_place(int j, int n, int lg) {
    const int lo = (int)(((uint64_t)j * (uint32_t)n) >> lg), hi = (int)(((uint64_t)(j + 1) * (uint32_t)n) >> lg);
    uint32_t h = (uint32_t)j * 0x9E3779B1u;
    h ^= h >> 15;
    h *= 0x85EBCA77u;
    h ^= h >> 13;
    return min(lo + (int)(((uint64_t)h * (uint32_t)max(1, hi - lo)) >> 32), n - 1);
}

__device__ __forceinline__ uint64_t depth_pair(uint32_t key, uint32_t val) { return ((uint64_t)key << 32) | val; }

// The samples' keys, for k_depth_bounds' workgroups to read side by side.
__global__ void __launch_bounds__(256) k_depth_samples(const uint32_t* __restrict__ keys, int n, int lg,
                                                       uint32_t* __restrict__ samples) {
    const int j = (int)(blockIdx.x * 256 + threadIdx.x);
    samples[((size_t)blockIdx.y << lg) + j] = keys[(size_t)blockIdx.y * n + sample_place(j, n, lg)];
}

// A workgroup ranks kSplitRanked samples against all: a sixteenth of them per wave,
// four at a time from LDS, the quarters of a wave side by side.  Every fourth sample
// in order is a bin's lower bound.  samples: their keys (null: read from keys by
// every workgroup).
constexpr int kSplitRanked = 16;
__global__ void __launch_bounds__(kSplitThreads) k_depth_bounds(const uint32_t* __restrict__ keys, uint32_t val0, int n,
                                                                int lg_bins, const uint32_t* __restrict__ samples,
                                                                uint64_t* __restrict__ bounds) {
    __shared__ __align__(16) uint32_t s_keys[kSplitOver * kSplitMaxBins];
    __shared__ uint32_t s_rank[kSplitThreads / 64][kSplitRanked];
    const int lg = lg_bins + 2, S = 1 << lg;  // (kSplitOver = 4)
    keys += (size_t)blockIdx.y * n;
    bounds += (size_t)blockIdx.y << lg_bins;
    if (samples) {
        const uint4* from = reinterpret_cast<const uint4*>(samples + ((size_t)blockIdx.y << lg));
        for (int j = threadIdx.x; j < S / 4; j += kSplitThreads) reinterpret_cast<uint4*>(s_keys)[j] = from[j];
    } else {
        for (int j = threadIdx.x; j < S; j += kSplitThreads) s_keys[j] = keys[sample_place(j, n, lg)];
    }
    __syncthreads();
    const int lane = __lane_id(), w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i0 = (int)blockIdx.x * kSplitRanked, i = i0 + lane % kSplitRanked;
    const uint32_t key = s_keys[i];
    const int j0 = w * (S / 16), j1 = j0 + S / 16;  // (multiples of 16)
    const int q = 4 * (lane / kSplitRanked);
    uint32_t r = 0u;
    const auto four = [&](int j) { return *reinterpret_cast<const uint4*>(&s_keys[j + q]); };
    // samples lie in id order: equal keys of lower index come before
    if (j1 <= i0) {
#pragma unroll 4
        for (int j = j0; j < j1; j += 16) {
            const uint4 k = four(j);
            r += (k.x <= key ? 1u : 0u) + (k.y <= key ? 1u : 0u) + (k.z <= key ? 1u : 0u) + (k.w <= key ? 1u : 0u);
        }
    } else if (j0 >= i0 + kSplitRanked) {
#pragma unroll 4
        for (int j = j0; j < j1; j += 16) {
            const uint4 k = four(j);
            r += (k.x < key ? 1u : 0u) + (k.y < key ? 1u : 0u) + (k.z < key ? 1u : 0u) + (k.w < key ? 1u : 0u);
        }
    } else {
        for (int j = j0; j < j1; j += 16) {
            const uint4 k = four(j);
            const int at = j + q;
            r += (k.x < key || (k.x == key && at < i) ? 1u : 0u) + (k.y < key || (k.y == key && at + 1 < i) ? 1u : 0u) +
                 (k.z < key || (k.z == key && at + 2 < i) ? 1u : 0u) + (k.w < key || (k.w == key && at + 3 < i) ? 1u : 0u);
        }
    }
    r += __shfl_xor(r, 16);
    r += __shfl_xor(r, 32);
    if (lane < kSplitRanked) s_rank[w][lane] = r;
    __syncthreads();
    if (threadIdx.x < kSplitRanked) {
        uint32_t at = 0u;
#pragma unroll
        for (int u = 0; u < kSplitThreads / 64; ++u) at += s_rank[u][lane];
        if (at > 0u && at % kSplitOver == 0u)
            bounds[at / kSplitOver - 1] = depth_pair(key, val0 + (uint32_t)sample_place(i, n, lg));
    }
}

// Counts of a workgroup's keys per bin (a row of 2^lg_bins), and each key's bin.
template <int ITEMS>
__global__ void __launch_bounds__(kSplitThreads) k_depth_count(const uint32_t* __restrict__ keys, uint32_t val0, int n,
                                                               int lg_bins, const uint64_t* __restrict__ bounds,
                                                               uint16_t* __restrict__ key_bin,
                                                               uint32_t* __restrict__ rows) {
    __shared__ uint64_t s_bound[kSplitMaxBins];
    __shared__ uint32_t s_count[kSplitMaxBins];
    const int tid = threadIdx.x, bins = 1 << lg_bins;
    const size_t seg = (size_t)blockIdx.y * n;
    const int begin = (int)blockIdx.x * (kSplitThreads * ITEMS);
    bounds += (size_t)blockIdx.y << lg_bins;
    uint64_t x[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = begin + k * kSplitThreads + tid;
        x[k] = depth_pair(i < n ? keys[seg + i] : 0u, val0 + (uint32_t)i);
    }
    for (int d = tid; d < bins; d += kSplitThreads) {
        s_bound[d] = d < bins - 1 ? bounds[d] : ~0ull;
        s_count[d] = 0u;
    }
    __syncthreads();
    int at[ITEMS];  // bounds at or below the key
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) at[k] = 0;
    for (int step = bins >> 1; step > 0; step >>= 1) {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) at[k] += s_bound[at[k] + step - 1] <= x[k] ? step : 0;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = begin + k * kSplitThreads + tid;
        if (i < n) {
            key_bin[seg + i] = (uint16_t)at[k];
            atomicAdd(&s_count[at[k]], 1u);
        }
    }
    __syncthreads();
    rows += ((size_t)blockIdx.y * gridDim.x + blockIdx.x) << lg_bins;
    for (int d = tid; d < bins; d += kSplitThreads) rows[d] = s_count[d];
}

// Exclusive scan of the rows down each bin's column, in place, and the totals: a
// workgroup takes 64 bins, each of its sixteen waves a sixteenth of the rows.
__global__ void __launch_bounds__(kSplitThreads) k_depth_columns(uint32_t* __restrict__ rows, int blocks, int lg_bins,
                                                                 uint32_t* __restrict__ totals) {
    __shared__ uint32_t s_sum[kSplitThreads / 64][64];
    const int lane = __lane_id(), w = (int)threadIdx.x >> 6, d = (int)blockIdx.x * 64 + lane;
    uint32_t* col = rows + (((size_t)blockIdx.y * blocks) << lg_bins) + d;
    const int per = (blocks + kSplitThreads / 64 - 1) / (kSplitThreads / 64);
    const int b0 = min(blocks, w * per), b1 = min(blocks, b0 + per);
    uint32_t sum = 0u;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) sum += col[(size_t)b << lg_bins];
    s_sum[w][lane] = sum;
    __syncthreads();
    uint32_t run = 0u, total = 0u;
#pragma unroll
    for (int q = 0; q < kSplitThreads / 64; ++q) {
        const uint32_t v = s_sum[q][lane];
        run += q < w ? v : 0u;
        total += v;
    }
    for (int b = b0; b < b1; b += 8) {
        uint32_t v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = b + q < b1 ? col[(size_t)(b + q) << lg_bins] : 0u;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (b + q < b1) col[(size_t)(b + q) << lg_bins] = run;
            run += v[q];
        }
    }
    if (w == 0) totals[((size_t)blockIdx.y << lg_bins) + d] = total;
}

// In-place exclusive scan of s[0 .. n), n <= 2048, by 1024 threads.
__device__ inline void block_scan_1024(uint32_t* s, int n, uint32_t* s_buf) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int per = n > kSplitThreads ? 2 : 1, d = tid * per;
    const uint32_t v0 = d < n ? s[d] : 0u, v1 = per == 2 ? s[d + 1] : 0u;
    uint32_t incl = v0 + v1;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) s_buf[w] = incl;
    __syncthreads();
    uint32_t run = incl - v0 - v1;
    for (int k = 0; k < w; ++k) run += s_buf[k];
    if (d < n) s[d] = run;
    if (per == 2) s[d + 1] = run + v0;
    __syncthreads();
}

// Keys to their bins (in any order inside), as pairs, through LDS so that a
// workgroup's keys of one bin are written together.
template <int ITEMS>
__global__ void __launch_bounds__(kSplitThreads) k_depth_scatter(const uint32_t* __restrict__ keys, uint32_t val0, int n,
                                                                 int lg_bins, const uint16_t* __restrict__ key_bin,
                                                                 const uint32_t* __restrict__ rows, int direct,
                                                                 const uint32_t* __restrict__ totals,
                                                                 uint32_t* __restrict__ starts,
                                                                 uint64_t* __restrict__ pairs) {
    constexpr int T = kSplitThreads * ITEMS;
    __shared__ uint64_t s_pair[T];
    __shared__ uint16_t s_bin[T];
    __shared__ uint32_t s_base[kSplitMaxBins], s_first[kSplitMaxBins];
    __shared__ uint32_t s_buf[kSplitThreads / 64];
    const int tid = threadIdx.x, bins = 1 << lg_bins, blocks = gridDim.x;
    const size_t seg = (size_t)blockIdx.y * n;
    const int begin = (int)blockIdx.x * T;
    uint32_t key[ITEMS];
    int bin[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = begin + k * kSplitThreads + tid;
        key[k] = i < n ? keys[seg + i] : 0u;
        bin[k] = i < n ? (int)key_bin[seg + i] : -1;
    }
    rows += ((size_t)blockIdx.y * blocks) << lg_bins;
    uint32_t before[kSplitMaxBins / kSplitThreads];
#pragma unroll
    for (int q = 0; q < kSplitMaxBins / kSplitThreads; ++q) {
        const int d = q * kSplitThreads + tid;
        before[q] = 0u;
        if (d >= bins) continue;
        uint32_t total = 0u;
        if (direct) {
            for (int b = 0; b < blocks; b += 16) {
                uint32_t v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) v[u] = b + u < blocks ? rows[((size_t)(b + u) << lg_bins) + d] : 0u;
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    total += v[u];
                    before[q] += b + u < (int)blockIdx.x ? v[u] : 0u;
                }
            }
        } else {
            total = totals[((size_t)blockIdx.y << lg_bins) + d];
            before[q] = rows[((size_t)blockIdx.x << lg_bins) + d];
        }
        s_base[d] = total;
        s_first[d] = 0u;
    }
    __syncthreads();
    uint32_t rank[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) rank[k] = bin[k] >= 0 ? atomicAdd(&s_first[bin[k]], 1u) : 0u;
    block_scan_1024(s_base, bins, s_buf);  // (its barriers also order the counts)
    block_scan_1024(s_first, bins, s_buf);
#pragma unroll
    for (int q = 0; q < kSplitMaxBins / kSplitThreads; ++q) {
        const int d = q * kSplitThreads + tid;
        if (d >= bins) continue;
        if (blockIdx.x == 0) starts[((size_t)blockIdx.y << lg_bins) + d] = s_base[d];
        s_base[d] += before[q] - s_first[d];
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        if (bin[k] < 0) continue;
        const uint32_t p = s_first[bin[k]] + rank[k];
        s_pair[p] = depth_pair(key[k], val0 + (uint32_t)(begin + k * kSplitThreads + tid));
        s_bin[p] = (uint16_t)bin[k];
    }
    __syncthreads();
    const int cnt = min(T, n - begin);
    for (int p = tid; p < cnt; p += kSplitThreads) pairs[seg + (uint32_t)(s_base[s_bin[p]] + (uint32_t)p)] = s_pair[p];
}

// The value of lane ^ J (14 of the 21 exchanges of a 64-lane sort stay in the
// vector unit).
template <int J>
__device__ __forceinline__ uint64_t lane_xor(uint64_t x) {
    if constexpr (J == 1 || J == 2 || J == 8) {
        constexpr int ctrl = J == 1 ? 0xB1 : J == 2 ? 0x4E : 0x128;  // quad_perm 1032, 2301; row_ror 8
        const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)x, ctrl, 0xF, 0xF, true);
        const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), ctrl, 0xF, 0xF, true);
        return depth_pair(hi, lo);
    } else {
        return __shfl_xor((unsigned long long)x, J);
    }
}
template <int K, int J>
__device__ __forceinline__ void lane_merge(uint64_t& x, int lane) {
    const uint64_t y = lane_xor<J>(x);
    const bool low = ((lane & J) == 0) == ((lane & K) == 0);
    x = (y < x) == low ? y : x;
    if constexpr (J > 1) lane_merge<K, J / 2>(x, lane);
}

// Runs of 64 of a block of m <= kBinKeys keys, each ordered among the lanes of one
// wave (padded with keys above all).
__device__ inline void bin_runs(const uint64_t* __restrict__ pairs, int m, uint64_t* s_run) {
    const int lane = __lane_id(), w = (int)threadIdx.x >> 6;
    for (int c = w; c * 64 < m; c += kBinWaves) {
        const int e = c * 64 + lane;
        uint64_t x = e < m ? pairs[e] : ~0ull;
        lane_merge<2, 1>(x, lane);
        lane_merge<4, 2>(x, lane);
        lane_merge<8, 4>(x, lane);
        lane_merge<16, 8>(x, lane);
        lane_merge<32, 16>(x, lane);
        lane_merge<64, 32>(x, lane);
        s_run[e] = x;
    }
}

// Keys below x in the runs [c0, c1).
__device__ __forceinline__ uint32_t runs_below(const uint64_t* s_run, int c0, int c1, uint64_t x) {
    uint32_t r = 0u;
#pragma unroll 4
    for (int c = c0; c < c1; ++c) {
        const uint64_t* run = s_run + c * 64;
        uint32_t at = 0u;
#pragma unroll
        for (int step = 32; step > 0; step >>= 1) at += run[at + step - 1] < x ? step : 0;
        r += at + (run[at] < x ? 1u : 0u);
    }
    return r;
}

// One bin in order: a key's place is its place in its run plus the keys below it in
// every other run.  A bin of more than kBinKeys keys goes block against block.
__global__ void __launch_bounds__(64 * kBinWaves) k_depth_bins(const uint64_t* __restrict__ pairs, int n, int lg_bins,
                                                    const uint32_t* __restrict__ starts, uint32_t* __restrict__ vals_out) {
    __shared__ uint64_t s_run[kBinKeys];
    const int bin = blockIdx.x, tid = threadIdx.x, lane = __lane_id(), w = tid >> 6;
    starts += (size_t)blockIdx.y << lg_bins;
    const int begin = (int)starts[bin], m = (bin + 1 < (1 << lg_bins) ? (int)starts[bin + 1] : n) - begin;
    pairs += (size_t)blockIdx.y * n + begin;
    vals_out += (size_t)blockIdx.y * n + begin;
    if (m <= kBinKeys) {
        bin_runs(pairs, m, s_run);
        __syncthreads();
        const int runs = (m + 63) / 64;
        for (int c = w; c < runs; c += kBinWaves) {
            const uint64_t x = s_run[c * 64 + lane];
            const uint32_t r = lane + runs_below(s_run, 0, c, x) + runs_below(s_run, c + 1, runs, x);
            if (c * 64 + lane < m) vals_out[r] = (uint32_t)x;
        }
        return;
    }
    constexpr int PER = kBinKeys / (64 * kBinWaves);
    for (int e0 = 0; e0 < m; e0 += kBinKeys) {
        uint64_t x[PER];
        uint32_t r[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = e0 + k * (64 * kBinWaves) + tid;
            x[k] = e < m ? pairs[e] : 0ull;
            r[k] = 0u;
        }
        for (int b = 0; b < m; b += kBinKeys) {
            const int mb = min(kBinKeys, m - b);
            __syncthreads();
            bin_runs(pairs + b, mb, s_run);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < PER; ++k) r[k] += runs_below(s_run, 0, (mb + 63) / 64, x[k]);
        }
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (e0 + k * (64 * kBinWaves) + tid < m) vals_out[r[k]] = (uint32_t)x[k];
    }
}

bool launch_depth_sort(uint32_t* keys, uint32_t val0, uint32_t* vals_out, int n, int n_seg, bool ranks,
                       uint64_t* pairs, uint32_t* work, size_t work_words, uint32_t* totals, size_t totals_words,
                       hipStream_t st) {
    if (n <= 0 || n_seg <= 0) return true;
    if (ranks) {
        k_rank_sort<<<dim3((unsigned)((n + 63) / 64), (unsigned)n_seg), 64 * kRankWaves, 0, st>>>(keys, val0, vals_out, n);
        return true;
    }
    const DepthPlan p = depth_plan(n, n_seg);
    if (p.words > work_words) return false;
    if (p.radix) {
        uint32_t* keys2 = reinterpret_cast<uint32_t*>(pairs);
        uint32_t* vals2 = keys2 + (size_t)n * n_seg;
        static_assert(32 % (2 * kDepthDigitBits) == 0, "the last pass ends in vals_out");
        for (int shift = 0; shift < 32; shift += kDepthDigitBits) {
            const bool odd = shift / kDepthDigitBits % 2 != 0;
            if (!launch_radix_pass(odd ? keys2 : keys, shift == 0 ? nullptr : odd ? vals2 : vals_out, odd ? keys : keys2,
                                   odd ? vals_out : vals2, nullptr, (uint64_t)n, (uint64_t)n, shift, kDepthDigitBits,
                                   work, work_words, totals, totals_words, nullptr, st, n_seg, (uint64_t)n, nullptr, 0,
                                   nullptr, 0, nullptr, nullptr, val0))
                return false;
        }
        return true;
    }
    const size_t bins = (size_t)1 << p.lg_bins;
    uint64_t* bounds = reinterpret_cast<uint64_t*>(work);
    uint32_t* counts = work + 2 * bins * n_seg;
    uint32_t* starts = counts + bins * n_seg;
    uint32_t* samples = starts + bins * n_seg;
    uint32_t* rows = samples + kSplitOver * bins * n_seg;
    uint16_t* key_bin = reinterpret_cast<uint16_t*>(vals_out);  // (until the bins are in order)
    const int direct = p.blocks <= kSplitDirect ? 1 : 0;
    const unsigned segs = (unsigned)n_seg;
    const dim3 grid((unsigned)p.blocks, segs);
    // (not by every workgroup that ranks some)
    const bool gather = kSplitOver * bins * n_seg >= kSplitGather;
    if (gather)
        k_depth_samples<<<dim3((unsigned)(kSplitOver * bins / 256), segs), 256, 0, st>>>(keys, n, p.lg_bins + 2, samples);
    k_depth_bounds<<<dim3((unsigned)(kSplitOver * bins / kSplitRanked), segs), kSplitThreads, 0, st>>>(
        keys, val0, n, p.lg_bins, gather ? samples : nullptr, bounds);
    if (p.items == 4)
        k_depth_count<4><<<grid, kSplitThreads, 0, st>>>(keys, val0, n, p.lg_bins, bounds, key_bin, rows);
    else
        k_depth_count<8><<<grid, kSplitThreads, 0, st>>>(keys, val0, n, p.lg_bins, bounds, key_bin, rows);
    if (!direct)
        k_depth_columns<<<dim3((unsigned)(bins / 64), segs), kSplitThreads, 0, st>>>(rows, p.blocks, p.lg_bins, counts);
    if (p.items == 4)
        k_depth_scatter<4><<<grid, kSplitThreads, 0, st>>>(keys, val0, n, p.lg_bins, key_bin, rows, direct, counts, starts,
                                                         pairs);
    else
        k_depth_scatter<8><<<grid, kSplitThreads, 0, st>>>(keys, val0, n, p.lg_bins, key_bin, rows, direct, counts, starts,
                                                         pairs);
    k_depth_bins<<<dim3((unsigned)bins, segs), 64 * kBinWaves, 0, st>>>(pairs, n, p.lg_bins, starts, vals_out);
    return true;
}

// ---------------------------------------------------------------------------
// 64-bit exclusive scan of (optionally gathered) 32-bit counts.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_scan_reduce(const uint32_t* __restrict__ in, const uint32_t* __restrict__ idx,
                                                     int n, unsigned long long* __restrict__ partials) {
    __shared__ unsigned long long s_buf[256];
    const int begin = blockIdx.x * kScanTile + threadIdx.x * 8;
    unsigned long long s = 0;
    for (int k = 0; k < 8; ++k) {
        const int i = begin + k;
        if (i < n) s += in[idx ? idx[i] : i];
    }
    unsigned long long tot;
    block_exclusive_scan_256<unsigned long long>(s, s_buf, tot);
    if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

// (blockIdx.x: the array; totals: where its total goes, null: behind it)
__global__ void __launch_bounds__(256) k_scan_top(unsigned long long* __restrict__ partials, int nparts, size_t stride,
                                                  unsigned long long* __restrict__ totals) {
    __shared__ unsigned long long s_buf[256];
    partials += (size_t)blockIdx.x * stride;
    unsigned long long carry = 0;
    for (int start = 0; start < nparts; start += 256) {
        const int i = start + threadIdx.x;
        const unsigned long long v = i < nparts ? partials[i] : 0ull;
        unsigned long long tot;
        const unsigned long long ex = block_exclusive_scan_256<unsigned long long>(v, s_buf, tot);
        if (i < nparts) partials[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) (totals ? totals[blockIdx.x] : partials[nparts]) = carry;
}

// With run_start: for every run of 256 outputs, the index whose range
// [out[i], out[i + 1]) holds the run's first output (runs below run_cap).
__global__ void __launch_bounds__(256) k_scan_down(const uint32_t* __restrict__ in, const uint32_t* __restrict__ idx,
                                                   int n, const unsigned long long* __restrict__ partials, int nparts,
                                                   unsigned long long* __restrict__ out,
                                                   uint32_t* __restrict__ run_start, uint64_t run_cap) {
    __shared__ unsigned long long s_buf[256];
    const int begin = blockIdx.x * kScanTile + threadIdx.x * 8;
    uint32_t v[8];
    unsigned long long s = 0;
    for (int k = 0; k < 8; ++k) {
        const int i = begin + k;
        v[k] = i < n ? in[idx ? idx[i] : i] : 0u;
        s += v[k];
    }
    unsigned long long tot;
    unsigned long long run = block_exclusive_scan_256<unsigned long long>(s, s_buf, tot) + partials[blockIdx.x];
    for (int k = 0; k < 8; ++k) {
        const int i = begin + k;
        if (i < n) {
            out[i] = run;
            if (run_start)
                for (uint64_t r = (run + 255) / 256; r * 256 < run + v[k] && r < run_cap; ++r) run_start[r] = (uint32_t)i;
        }
        run += v[k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = partials[nparts];
}

int scan_blocks(int n) { return (int)(((int64_t)n + kScanTile - 1) / kScanTile); }

void launch_scan_top(unsigned long long* partials, int nparts, int count, size_t stride, unsigned long long* totals,
                     hipStream_t st) {
    k_scan_top<<<count, 256, 0, st>>>(partials, nparts, stride, totals);
}

void launch_scan_u32_u64(const uint32_t* in, const uint32_t* idx, int n, unsigned long long* out,
                         unsigned long long* partials, hipStream_t st, uint32_t* run_start, uint64_t run_cap) {
    const int nb = std::max(1, scan_blocks(n));
    k_scan_reduce<<<nb, 256, 0, st>>>(in, idx, n, partials);
    k_scan_top<<<1, 256, 0, st>>>(partials, nb, 0, nullptr);
    k_scan_down<<<nb, 256, 0, st>>>(in, idx, n, partials, nb, out, run_start, run_cap);
}

// ---------------------------------------------------------------------------
// Two-level binning.
// ---------------------------------------------------------------------------
__host__ __device__ __forceinline__ uint64_t pack_rect(uint32_t x0, uint32_t x1, uint32_t y0, uint32_t y1) {
    return (uint64_t)x0 | ((uint64_t)x1 << 16) | ((uint64_t)y0 << 32) | ((uint64_t)y1 << 48);
}

// Flags in the top bits of a splat's packed tile rectangle (tile coordinates
// stay below 2^14): the shape test per coarse entry, or no test at all; both
// for a splat without entries.
constexpr uint64_t kRectShape = 1ull << 63, kRectFull = 1ull << 62;
constexpr uint64_t kRectNone = kRectShape | kRectFull, kRectCoords = ~kRectNone;

// Where depth-ordered entry j of a pass (segment layout sg) belongs: the view
// whose records hold it and, for its super-tile keys, that view's grid and the
// grid's first super-tile id relative to the pass (a static group's grid for
// the group segments).
struct SegPos {
    int view, super0;
};
__device__ __forceinline__ SegPos seg_of(int j, const SegLayout& sg, const ViewParams* __restrict__ views, int v0) {
    const int split = sg.na * sg.la;
    if (j < split) {
        const int v = v0 + j / sg.la;
        return SegPos{v, views[v].super_base - views[v0].super_base};
    }
    const int leader = views[(j - split) / sg.lb].group_leader;
    return SegPos{leader, views[leader].static_super_base - views[v0].super_base};
}

// Tiles of the super-tile at tile origin (bx, by) in the tabulated spans of
// rows [ty0, ty1] (span_row[row - ty0]), as tile_mask's bits.
template <int TILE>
__host__ __device__ inline uint32_t span_mask(const uint32_t* span_row, uint32_t ty0, uint32_t ty1, uint32_t bx,
                                              uint32_t by) {
    constexpr uint32_t S = (uint32_t)super_factor(TILE);
    uint32_t m = 0u;
#pragma unroll
    for (uint32_t ly = 0; ly < S; ++ly) {
        const uint32_t ty = by + ly;
        if (ty < ty0 || ty > ty1) continue;
        const uint32_t e = span_row[ty - ty0];
        const uint32_t lo = (e & 0xFFFFu) > bx ? (e & 0xFFFFu) : bx, hi = (e >> 16) < bx + S ? (e >> 16) : bx + S;
        if (lo < hi) m |= ((1u << (hi - bx)) - (1u << (lo - bx))) << (ly * S);
    }
    return m;
}

// Where block b of a binning pass lies (blocks never straddle segments): its
// segment, the block's number in it, its depth-ordered entries [j0, j0 + n),
// the view whose records they index, that segment's super-tiles and the first
// global super-tile id of its grid.
struct BinBlock {
    int seg, block, j0, n, view, sx, supers, super_base;
};
__device__ __forceinline__ BinBlock bin_block(int b, const SegLayout& sg, const ViewParams* __restrict__ views, int v0) {
    BinBlock r;
    const int nba = ceil_div(sg.la, kBinBlock), nbb = ceil_div(sg.lb, kBinBlock);
    int len;
    if (b < sg.na * nba) {
        r.seg = b / nba;
        r.block = b - r.seg * nba;
        r.j0 = r.seg * sg.la;
        len = sg.la;
        r.view = v0 + r.seg;
        r.super_base = views[r.view].super_base;
    } else {
        const int g = (b - sg.na * nba) / nbb;
        r.seg = sg.na + g;
        r.block = b - sg.na * nba - g * nbb;
        r.j0 = sg.na * sg.la + g * sg.lb;
        len = sg.lb;
        r.view = views[g].group_leader;
        r.super_base = views[r.view].static_super_base;
    }
    r.j0 += r.block * kBinBlock;
    r.n = min(kBinBlock, len - r.block * kBinBlock);
    r.sx = views[r.view].sx;
    r.supers = r.sx * views[r.view].sy;
    return r;
}

// Per depth-ordered entry j of the pass: its tile rectangle and its
// super-tile count.  With culling (shapes != null) the rectangle shrinks to
// the rows whose slab meets the ellipse and to the columns any of their spans
// keeps (the tiles tile_mask can keep; a splat with none emits nothing), and
// the spans of up to kSpanRows rows are tabulated for the emission
// (spans[j * kSpanRows + row - first row]); a taller splat keeps its shape
// (kRectShape: tested per entry) and one without a proper ellipse its square
// (kRectFull: untested).  The spans of a wave's splats are computed one
// (splat, row) per lane: a wave's rows are numbered by a prefix sum over its
// lanes, and each round of 64 finds its rows' splats by a max-scan of the
// lanes' first rows.
// One entry per thread; each workgroup also leaves its sum of counts for
// the offsets' scan (partials[blockIdx.x]).
template <int TILE>
__global__ void __launch_bounds__(256, 6) k_coarse_count(const uint32_t* __restrict__ sorted_gid, int n, int N,
                                                      SegLayout sg, const Rec* __restrict__ recs,
                                                      const ViewParams* __restrict__ views, int v0,
                                                      uint32_t* __restrict__ cnt, uint64_t* __restrict__ rect_sorted,
                                                      CullShape* __restrict__ shapes, uint32_t* __restrict__ spans,
                                                      unsigned long long* __restrict__ partials) {
    constexpr uint32_t S = (uint32_t)super_factor(TILE);
    __shared__ unsigned long long s_buf[256];
    __shared__ CullShape s_cs[256];
    __shared__ int s_cmin[256], s_cmax[256];
    __shared__ int s_slot[4][64];
    const int tid = (int)threadIdx.x, lane = __lane_id(), w = tid >> 6;
    const int j = blockIdx.x * 256 + tid;
    bool keep = false;
    uint64_t flags = 0ull;
    int tx0 = 0, tx1 = -1, ty0 = 0, ty1 = -1, r0 = 0, nrows = 0;
    if (j < n) {
        const SegPos sp = seg_of(j, sg, views, v0);
        const Rec& rec = recs[(size_t)sp.view * N + sorted_gid[j]];
        const uint4 d = rec.d;
        if (d.w != 0u) {
            keep = true;
            tx0 = (int)((d.x & 0xFFFFu) / TILE); tx1 = (int)((d.x >> 16) / TILE);
            ty0 = (int)((d.y & 0xFFFFu) / TILE); ty1 = (int)((d.y >> 16) / TILE);
            if (shapes) {
                const CullShape cs = cull_shape(rec);
                if (cs.mode == 0) {
                    flags = kRectFull;
                } else if (cs.mode == 2) {
                    keep = false;
                } else {
                    int r1;
                    slab_rows<TILE>(cs, ty0, ty1, r0, r1);
                    nrows = max(0, r1 - r0 + 1);
                    keep = nrows > 0;
                    s_cs[tid] = cs;
                }
            }
        }
    }
    if (shapes) {  // uniform
        s_cmin[tid] = tx1 + 1;
        s_cmax[tid] = tx0 - 1;
        int incl = nrows;
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(incl, off);
            if (lane >= off) incl += y;
        }
        const int total = __shfl(incl, 63), excl = incl - nrows;
        const bool table = nrows <= kSpanRows;
        int carry = 0;  // the lane whose rows hold the round's first
        for (int base = 0; base < total; base += 64) {
            s_slot[w][lane] = -1;
            __builtin_amdgcn_wave_barrier();
            if (nrows > 0 && excl >= base && excl < base + 64) s_slot[w][excl - base] = lane;
            __builtin_amdgcn_wave_barrier();
            int o = s_slot[w][lane];
            if (lane == 0 && o < 0) o = carry;
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(o, off);
                if (lane >= off) o = max(o, y);
            }
            carry = __shfl(o, 63);
            const int g = max(o, 0);
            const int ex = __shfl(excl, g), gr0 = __shfl(r0, g), gx0 = __shfl(tx0, g), gx1 = __shfl(tx1, g);
            const int gtab = __shfl((int)table, g);
            const int k = base + lane;
            if (k < total) {
                const int gt = (w << 6) + g;
                const uint32_t e = row_columns<TILE>(s_cs[gt], gr0 + (k - ex), gx0, gx1);
                if (gtab) spans[((size_t)blockIdx.x * 256 + gt) * kSpanRows + (k - ex)] = e;
                if (e != 0u) {
                    atomicMin(&s_cmin[gt], (int)(e & 0xFFFFu));
                    atomicMax(&s_cmax[gt], (int)(e >> 16) - 1);
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        if (keep && nrows > 0) {
            const int cmin = s_cmin[tid], cmax = s_cmax[tid];
            keep = cmin <= cmax;
            if (keep) {
                tx0 = cmin; tx1 = cmax; ty0 = r0; ty1 = r0 + nrows - 1;
                if (!table) {
                    flags = kRectShape;
                    shapes[j] = s_cs[tid];
                }
            }
        }
    }
    uint32_t c = 0u;
    if (j < n) {
        uint64_t rect = 0ull;
        if (keep) {
            rect = pack_rect((uint32_t)tx0, (uint32_t)tx1, (uint32_t)ty0, (uint32_t)ty1) | flags;
            c = ((uint32_t)tx1 / S - (uint32_t)tx0 / S + 1u) * ((uint32_t)ty1 / S - (uint32_t)ty0 / S + 1u);
        }
        rect_sorted[j] = rect;
        cnt[j] = c;
    }
    unsigned long long tot;
    block_exclusive_scan_256<unsigned long long>((unsigned long long)c, s_buf, tot);
    if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

// Counting variant only: (view, Gaussian) pairs of the views [v0, v0 + nv)
// whose pixel square meets the image (the on-screen pairs; a 3D Gaussian's
// record is its view's static_view's), added to *counter.  grid.y: the view.
__global__ void __launch_bounds__(256) k_count_onscreen(const Rec* __restrict__ recs, int N, int n4,
                                                        const ViewParams* __restrict__ views, int v0,
                                                        unsigned long long* counter) {
    const int i = blockIdx.x * 256 + (int)threadIdx.x;
    const int v = v0 + (int)blockIdx.y;
    const int rv = i < n4 ? v : views[v].static_view;
    const bool on = i < N && recs[(size_t)rv * N + i].d.w != 0u;
    const unsigned long long c = (unsigned long long)__popcll(__ballot(on));
    if (__lane_id() == 0 && c) atomicAdd(counter, c);
}

void launch_count_onscreen(const Rec* recs, int N, int n4, const ViewParams* views, int v0, int nv,
                           unsigned long long* counter, hipStream_t st) {
    if (N == 0 || nv == 0) return;
    k_count_onscreen<<<dim3((unsigned)((N + 255) / 256), nv), 256, 0, st>>>(recs, N, n4, views, v0, counter);
}

// offsets[j] = partials[j / 256] (scanned) + this workgroup's exclusive scan;
// run_start as in k_scan_down.
__global__ void __launch_bounds__(256) k_coarse_down(const uint32_t* __restrict__ cnt, int n,
                                                     const unsigned long long* __restrict__ partials, int nparts,
                                                     unsigned long long* __restrict__ offsets,
                                                     uint32_t* __restrict__ run_start, uint64_t run_cap) {
    __shared__ unsigned long long s_buf[256];
    const int j = blockIdx.x * 256 + (int)threadIdx.x;
    const uint32_t c = j < n ? cnt[j] : 0u;
    unsigned long long tot;
    const unsigned long long run =
        block_exclusive_scan_256<unsigned long long>((unsigned long long)c, s_buf, tot) + partials[blockIdx.x];
    if (j < n) {
        offsets[j] = run;
        for (uint64_t r = (run + 255) / 256; r * 256 < run + c && r < run_cap; ++r) run_start[r] = (uint32_t)j;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) offsets[n] = partials[nparts];
}

// The capacity check of a pass whose coarse entries total C (one thread): its
// entries take [cbase[v0], cbase[v0] + C) of the call's ccap; the need is
// counted in (Gaussian, tile) slots, S^2 per coarse entry.
__device__ inline void coarse_finalize(unsigned long long C, uint64_t ccap, int S, unsigned long long* cbase, int v0,
                                       int v1, Status* status, unsigned long long* eff_count) {
    const unsigned long long base = cbase[v0];
    status->pairs_needed += C * (unsigned long long)(S * S);
    if (base + C > ccap) {
        status->flags |= kFlagOverflow;
        *eff_count = 0ull;
        cbase[v1] = base;
    } else {
        *eff_count = C;
        cbase[v1] = base + C;
    }
}

// Few count workgroups (nparts <= kDirectParts): k_coarse_top and k_coarse_down
// in one launch.  Each workgroup sums the partials of the workgroups before it
// (workgroup 0 sums them all, finalizes the pass and writes offsets[n]), then
// scans its own counts as k_coarse_down does.
constexpr int kDirectParts = 2048;
__global__ void __launch_bounds__(256) k_coarse_down_direct(const uint32_t* __restrict__ cnt, int n,
                                                            const unsigned long long* __restrict__ partials,
                                                            int nparts, uint64_t ccap, int S,
                                                            unsigned long long* cbase, int v0, int v1,
                                                            Status* status, unsigned long long* eff_count,
                                                            unsigned long long* __restrict__ offsets,
                                                            uint32_t* __restrict__ run_start, uint64_t run_cap) {
    __shared__ unsigned long long s_buf[256];
    const int b = (int)blockIdx.x;
    const int upto = b == 0 ? nparts : b;
    unsigned long long acc = 0;
    for (int i = (int)threadIdx.x; i < upto; i += 256) acc += partials[i];
    unsigned long long sum;
    block_exclusive_scan_256<unsigned long long>(acc, s_buf, sum);
    const unsigned long long before = b == 0 ? 0ull : sum;
    if (b == 0 && threadIdx.x == 0) {
        coarse_finalize(sum, ccap, S, cbase, v0, v1, status, eff_count);
        offsets[n] = sum;
    }
    const int j = b * 256 + (int)threadIdx.x;
    const uint32_t c = j < n ? cnt[j] : 0u;
    unsigned long long tot;
    const unsigned long long run = block_exclusive_scan_256<unsigned long long>((unsigned long long)c, s_buf, tot) + before;
    if (j < n) {
        offsets[j] = run;
        for (uint64_t r = (run + 255) / 256; r * 256 < run + c && r < run_cap; ++r) run_start[r] = (uint32_t)j;
    }
}

// Exclusive scan of the count workgroups' sums (partials[nparts] = total C),
// then the coarse capacity check of the pass (coarse_finalize).
// (1024 threads, each scanning a contiguous chunk of the partials four loads
// at a time: with many count workgroups, e.g. 32 views of 1M Gaussians, this
// single workgroup's walk over the partials is the launch)
__global__ void __launch_bounds__(1024) k_coarse_top(unsigned long long* __restrict__ partials, int nparts,
                                                     uint64_t ccap, int S, unsigned long long* cbase, int v0,
                                                     int v1, Status* status, unsigned long long* eff_count) {
    __shared__ unsigned long long s_w[16];
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    // thread t scans the contiguous chunk [t q, (t + 1) q) of the partials
    const int q = (nparts + 1023) / 1024;
    const int i0 = min(nparts, tid * q), i1 = min(nparts, i0 + q);
    unsigned long long a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    int i = i0;
    for (; i + 3 < i1; i += 4) {
        a0 += partials[i];
        a1 += partials[i + 1];
        a2 += partials[i + 2];
        a3 += partials[i + 3];
    }
    for (; i < i1; ++i) a0 += partials[i];
    const unsigned long long sum = (a0 + a1) + (a2 + a3);
    // exclusive scan of the chunk sums over the workgroup (wave scans, then the
    // 16 wave totals)
    unsigned long long incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) s_w[w] = incl;
    __syncthreads();
    unsigned long long run = incl - sum, carry = 0;
    for (int k = 0; k < 16; ++k) {
        const unsigned long long t = s_w[k];
        if (k < w) run += t;
        carry += t;
    }
    for (i = i0; i + 3 < i1; i += 4) {
        const unsigned long long v0_ = partials[i], v1_ = partials[i + 1], v2_ = partials[i + 2], v3_ = partials[i + 3];
        partials[i] = run;
        partials[i + 1] = run + v0_;
        partials[i + 2] = run + v0_ + v1_;
        partials[i + 3] = run + v0_ + v1_ + v2_;
        run += v0_ + v1_ + v2_ + v3_;
    }
    for (; i < i1; ++i) {
        const unsigned long long v = partials[i];
        partials[i] = run;
        run += v;
    }
    if (tid != 0) return;
    partials[nparts] = carry;
    coarse_finalize(carry, ccap, S, cbase, v0, v1, status, eff_count);
}

// Coarse entries (super-tile id relative to the pass's first, depth rank j),
// written in (segment, depth) order: one thread per entry, which finds its
// Gaussian by binary search over the count offsets (entries, not Gaussians,
// are spread evenly: the nearest splats are the largest and sit together in
// depth order).  The key's upper 16 bits carry the entry's tile mask (the
// super-tile sort reads only the low bits); shapes != null applies the alpha
// >= 1/255 tile test.
template <int TILE>
__global__ void __launch_bounds__(256) k_coarse_emit(const unsigned long long* __restrict__ offsets,
                                                     const uint32_t* __restrict__ run_start, int n, SegLayout sg,
                                                     const uint64_t* __restrict__ rect_sorted,
                                                     const CullShape* __restrict__ shapes,
                                                     const uint32_t* __restrict__ spans,
                                                     const ViewParams* __restrict__ views, int v0,
                                                     const unsigned long long* eff_count,
                                                     uint32_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    constexpr uint32_t S = (uint32_t)super_factor(TILE);
    __shared__ unsigned long long s_off[257];
    const uint64_t C = *eff_count;
    const int tid = threadIdx.x;
    // blocks take runs of 256 consecutive entries (run_start names the Gaussian
    // holding a run's first entry); within a segment invisible
    // Gaussians sort last (culled key), so the visible ones all own entries and
    // a run usually spans at most 256 consecutive Gaussians (entries past the
    // block's window, after another segment's invisible tail, search globally)
    for (uint64_t p0 = (uint64_t)blockIdx.x * 256; p0 < C; p0 += (uint64_t)gridDim.x * 256) {
        const int j0 = (int)run_start[p0 / 256];  // Gaussian holding entry p0
        s_off[tid] = offsets[min(j0 + tid, n)];
        if (tid == 0) s_off[256] = offsets[min(j0 + 256, n)];
        __syncthreads();
        const uint64_t p = p0 + tid;
        if (p < C) {
            int j;
            unsigned long long pj;  // offsets[j]
            if (p < s_off[256]) {
                int lo = 0, hi = 256;  // last k with s_off[k] <= p
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_off[mid] <= p) lo = mid; else hi = mid;
                }
                j = j0 + lo;
                pj = s_off[lo];
            } else {
                int lo = min(j0 + 256, n - 1), hi = n;  // offsets[lo] <= p < offsets[n]
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (offsets[mid] <= p) lo = mid; else hi = mid;
                }
                j = lo;
                pj = offsets[lo];
            }
            const SegPos sp = seg_of(j, sg, views, v0);
            const ViewParams& V = views[sp.view];
            const uint64_t rf = rect_sorted[j], r = rf & kRectCoords;
            const uint32_t tx0 = (uint32_t)(r & 0xFFFFu), tx1 = (uint32_t)((r >> 16) & 0xFFFFu);
            const uint32_t ty0 = (uint32_t)((r >> 32) & 0xFFFFu), ty1 = (uint32_t)(r >> 48);
            const uint32_t sx0 = tx0 / S, sw = tx1 / S - sx0 + 1u, sy0 = ty0 / S;
            // (row, column) of the entry in the splat's sw-wide block of
            // super-tiles: a float quotient, exact after one correction
            // (local < 2^24)
            const uint32_t local = (uint32_t)(p - pj);
            uint32_t sy = (uint32_t)((float)local * __builtin_amdgcn_rcpf((float)sw));
            if (sy * sw > local) --sy;
            else if ((sy + 1u) * sw <= local) ++sy;
            const uint32_t sx = local - sy * sw;
            uint32_t key = (uint32_t)sp.super0 + (sy0 + sy) * (uint32_t)V.sx + sx0 + sx;
            const uint32_t bx = (sx0 + sx) * S, by = (sy0 + sy) * S;
            uint32_t m;
            if (!shapes || (rf & kRectFull)) {
                m = tile_mask<TILE>(CullShape{}, false, tx0, tx1, ty0, ty1, bx, by);
            } else if (rf & kRectShape) {
                m = tile_mask<TILE>(shapes[j], true, tx0, tx1, ty0, ty1, bx, by);
            } else {
                m = span_mask<TILE>(spans + (size_t)j * kSpanRows, ty0, ty1, bx, by);
            }
            key |= m << 16;
            keys[p] = key;
            vals[p] = (uint32_t)j;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Ranked binning: the coarse lists without a sort.
// ---------------------------------------------------------------------------
// A block of kBinBlock depth-ordered splats sets, per super-tile of the view,
// one bit per splat that reaches it; the rank of a splat's entry within the
// block's run of that super-tile's list is the number of set bits below its
// own, so that the entries go straight to their place in depth order.  The
// runs' starts come from the blocks' histograms (k_bin_count),
// scanned over the blocks in two levels.  Against emitting the entries and
// sorting them stably by super-tile, each entry is written once instead of two
// or three times and read by no sort pass.

// Item p of a wave's SPLATS splats: one row of super-tiles of one splat (pre: the
// exclusive prefix of the splats' row counts; rects: their packed tile
// rectangles, rows as the slab test left them).
struct BinItem {
    int g;          // the splat's lane
    uint32_t row;   // the row of super-tiles
    uint32_t slot;  // its number among the splat's
    uint32_t tx0, tx1, ty0, ty1;
    uint64_t flags;
};
template <int TILE, int SPLATS>
__device__ __forceinline__ BinItem bin_item(uint32_t p, const uint32_t* pre, const uint64_t* rects) {
    constexpr uint32_t S = (uint32_t)super_factor(TILE);
    int g = 0;
#pragma unroll
    for (int st = SPLATS / 2; st > 0; st >>= 1)
        if (pre[g + st] <= p) g += st;  // the last splat that starts at or before p (one with rows)
    const uint64_t r = rects[g];
    BinItem it;
    it.g = g;
    it.flags = r & kRectNone;
    it.tx0 = (uint32_t)(r & 0xFFFFu);
    it.tx1 = (uint32_t)((r >> 16) & 0xFFFFu);
    it.ty0 = (uint32_t)((r >> 32) & 0xFFFFu);
    it.ty1 = (uint32_t)(r >> 48) & 0x3FFFu;
    it.slot = p - pre[g];
    it.row = it.ty0 / S + it.slot;
    return it;
}
// Rows of super-tiles of a packed tile rectangle (0 without entries).
template <int TILE>
__device__ __forceinline__ uint32_t bin_rows(uint64_t r) {
    constexpr uint32_t S = (uint32_t)super_factor(TILE);
    if ((r & kRectNone) == kRectNone) return 0u;
    return ((uint32_t)(r >> 48) & 0x3FFFu) / S - ((uint32_t)(r >> 32) & 0xFFFFu) / S + 1u;
}
// The column spans (first | (last + 1) << 16, 0: none) of an item's tile rows:
// the whole rectangle's, or, with a shape, those the ellipse keeps.
template <int TILE>
__device__ __forceinline__ void item_spans(const BinItem& it, const CullShape* cs, uint32_t e[super_factor(TILE)]) {
    constexpr uint32_t S = (uint32_t)super_factor(TILE);
#pragma unroll
    for (uint32_t q = 0; q < S; ++q) {
        const uint32_t y = it.row * S + q;
        e[q] = 0u;
        if (y >= it.ty0 && y <= it.ty1)
            e[q] = cs ? row_columns<TILE>(*cs, (int)y, (int)it.tx0, (int)it.tx1) : it.tx0 | ((it.tx1 + 1u) << 16);
    }
}
// First and last tile column of the item's spans (c0 > c1: none).  The item's
// entries are the super-tiles between them: the spans of an ellipse's rows
// adjoin, so that one between them with an empty mask is rare, and harmless.
template <int TILE>
__device__ __forceinline__ void item_columns(const uint32_t e[super_factor(TILE)], uint32_t& c0, uint32_t& c1) {
    c0 = 0xFFFFu;
    c1 = 0u;
#pragma unroll
    for (int q = 0; q < super_factor(TILE); ++q)
        if (e[q] != 0u) {
            c0 = min(c0, e[q] & 0xFFFFu);
            c1 = max(c1, (e[q] >> 16) - 1u);
        }
}

// Rows of super-tiles whose spans are tabulated per splat (8 bytes each: a
// first column and an end per tile row, relative to the splat's first tile
// column); a splat with more rows, or wider than a byte's columns, keeps its
// shape (kRectShape) and its spans are found again by the scatter.
constexpr int kBinSlots = 4 * kSpanRows / 8;
constexpr int kBinWide = 255;

// Per depth-ordered entry of a block: its tile rectangle (the rows whose slab
// meets the ellipse), the spans of its rows of super-tiles (one per lane and
// round, a wave's rows numbered by a prefix sum over its splats), and per
// super-tile of the grid the block's entries: row blockIdx.x of hist, `words`
// words of two 16-bit counts.  partials: the block's entries over the splats'
// shrunk rectangles, which the capacity counts.
// Bound by instruction issue: each lane finds its four rows' spans with two
// roots per row and integer ends (row_columns); stepping the ends to the exact
// float comparisons tile by tile took 0.044 instead of 0.023 ms (250k splats, 1352 x
// 1014) and 0.151 instead of 0.067 ms (1M, 2704 x 2028).
template <int TILE>
__global__ void __launch_bounds__(256) k_bin_count(const uint32_t* __restrict__ sorted_gid, int N, SegLayout sg,
                                                   const Rec* __restrict__ recs, const ViewParams* __restrict__ views,
                                                   int v0, uint64_t* __restrict__ rect_sorted,
                                                   CullShape* __restrict__ shapes, uint2* __restrict__ spans,
                                                   unsigned long long* __restrict__ partials,
                                                   uint32_t* __restrict__ hist, int words) {
    constexpr uint32_t S = (uint32_t)super_factor(TILE);
    __shared__ CullShape s_cs[256];
    __shared__ int s_cmin[256], s_cmax[256];
    __shared__ uint32_t s_pre[256];
    __shared__ uint64_t s_rect[256];
    __shared__ unsigned long long s_buf[256];
    extern __shared__ uint32_t s_count[];  // the block's counts, two per word
    const int tid = (int)threadIdx.x, lane = __lane_id(), w0 = tid & ~63;
    const BinBlock bb = bin_block((int)blockIdx.x, sg, views, v0);
    const int j = bb.j0 + tid;
    for (int k = tid; k < words; k += 256) s_count[k] = 0u;
    uint64_t rect = kRectNone;
    int mode = 0;
    if (tid < bb.n) {
        const Rec& rec = recs[(size_t)bb.view * N + sorted_gid[j]];
        const uint4 d = rec.d;
        if (d.w != 0u) {
            int tx0 = (int)((d.x & 0xFFFFu) / TILE), tx1 = (int)((d.x >> 16) / TILE);
            int ty0 = (int)((d.y & 0xFFFFu) / TILE), ty1 = (int)((d.y >> 16) / TILE);
            uint64_t flags = 0ull;
            if (shapes) {
                const CullShape cs = cull_shape(rec);
                mode = cs.mode;
                if (mode == 1) {
                    int r0, r1;
                    slab_rows<TILE>(cs, ty0, ty1, r0, r1);
                    if (r1 < r0) {
                        mode = 2;
                    } else {
                        ty0 = r0;
                        ty1 = r1;
                        if (ty1 / (int)S - ty0 / (int)S >= kBinSlots || tx1 - tx0 >= kBinWide) flags = kRectShape;
                        s_cs[tid] = cs;
                        if (flags) shapes[j] = cs;
                    }
                }
            }
            if (mode == 0) flags = kRectFull;
            if (mode != 2) rect = pack_rect((uint32_t)tx0, (uint32_t)tx1, (uint32_t)ty0, (uint32_t)ty1) | flags;
        }
    }
    s_cmin[tid] = 0xFFFF;
    s_cmax[tid] = -1;
    const uint32_t rows = bin_rows<TILE>(rect);
    uint32_t incl = rows;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    s_pre[tid] = incl - rows;
    s_rect[tid] = rect;
    const uint32_t total = __shfl(incl, 63);
    __syncthreads();
    for (uint32_t p = (uint32_t)lane; p < total; p += 64) {
        const BinItem it = bin_item<TILE, 64>(p, s_pre + w0, s_rect + w0);
        const int gt = w0 + it.g;
        uint32_t e[S], c0, c1;
        item_spans<TILE>(it, it.flags == kRectFull ? nullptr : &s_cs[gt], e);
        item_columns<TILE>(e, c0, c1);
        if (it.flags == 0ull) {  // the table (a row without columns: both bytes 0)
            uint32_t b[2] = {0u, 0u};
#pragma unroll
            for (uint32_t q = 0; q < S; ++q)
                if (e[q] != 0u)
                    b[q >> 1] |= (((e[q] & 0xFFFFu) - it.tx0) | (((e[q] >> 16) - it.tx0) << 8)) << (16 * (q & 1u));
            spans[((size_t)bb.j0 + gt) * kBinSlots + it.slot] = make_uint2(b[0], b[1]);
        }
        if (c0 > c1) continue;
        atomicMin(&s_cmin[gt], (int)c0);
        atomicMax(&s_cmax[gt], (int)c1);
        const uint32_t at = it.row * (uint32_t)bb.sx;
        for (uint32_t t = at + c0 / S; t <= at + c1 / S; ++t) atomicAdd(&s_count[t >> 1], (t & 1u) ? 0x10000u : 1u);
    }
    __syncthreads();
    uint32_t c = 0u;
    const int cmin = s_cmin[tid], cmax = s_cmax[tid];
    if (cmin <= cmax) c = ((uint32_t)cmax / S - (uint32_t)cmin / S + 1u) * rows;
    if (tid < bb.n) rect_sorted[j] = c == 0u ? kRectNone : rect;
    for (int k = tid; k < words; k += 256) hist[(size_t)blockIdx.x * words + k] = s_count[k];
    unsigned long long tot;
    block_exclusive_scan_256<unsigned long long>((unsigned long long)c, s_buf, tot);
    if (tid == 0) partials[blockIdx.x] = tot;
}

// In place: hist rows become, within each chunk of kBinChunk blocks of one
// segment, the exclusive sums over the chunk's blocks before; chunk_sums[chunk]
// [2 words] the chunk's totals.  Two 16-bit counts share a word: a chunk's
// total is at most 64 x 256.  grid: a workgroup per chunk and 64 words, the chunk's
// side by side (in x, where more than 65535 chunks fit as well).
__global__ void __launch_bounds__(256) k_bin_chunks(uint32_t* __restrict__ hist, int words, SegLayout sg,
                                                    const unsigned long long* __restrict__ partials,
                                                    uint2* __restrict__ chunk_sums,
                                                    unsigned long long* __restrict__ chunk_entries) {
    __shared__ uint32_t s_sum[4][64];
    const int nba = ceil_div(sg.la, kBinBlock), nbb = ceil_div(sg.lb, kBinBlock);
    const int nca = ceil_div(nba, kBinChunk), ncb = ceil_div(nbb, kBinChunk);
    const int cols = ceil_div(words, 64), c = (int)blockIdx.x / cols, col0 = (int)blockIdx.x - c * cols;
    int b0, nb;  // the chunk's blocks
    if (c < sg.na * nca) {
        const int s = c / nca, k = c - s * nca;
        b0 = s * nba + k * kBinChunk;
        nb = min(kBinChunk, nba - k * kBinChunk);
    } else {
        const int s = (c - sg.na * nca) / ncb, k = c - sg.na * nca - s * ncb;
        b0 = sg.na * nba + s * nbb + k * kBinChunk;
        nb = min(kBinChunk, nbb - k * kBinChunk);
    }
    const int col = col0 * 64 + ((int)threadIdx.x & 63), rg = (int)threadIdx.x >> 6;
    constexpr int R = kBinChunk / 4;
    uint32_t v[R], sum = 0u;
    uint32_t* h = hist + (size_t)(b0 + rg * R) * words + col;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        v[r] = (col < words && rg * R + r < nb) ? h[(size_t)r * words] : 0u;
        sum += v[r];
    }
    s_sum[rg][threadIdx.x & 63] = sum;
    __syncthreads();
    uint32_t run = 0u, total = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t t = s_sum[q][threadIdx.x & 63];
        if (q < rg) run += t;
        total += t;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (col < words && rg * R + r < nb) h[(size_t)r * words] = run;
        run += v[r];
    }
    if (rg == 0 && col < words) chunk_sums[(size_t)c * words + col] = make_uint2(total & 0xFFFFu, total >> 16);
    if (col0 == 0 && threadIdx.x < 64) {
        unsigned long long e = (int)threadIdx.x < nb ? partials[b0 + threadIdx.x] : 0ull;
        for (int off = 32; off > 0; off >>= 1) e += (unsigned long long)__shfl_xor((long long)e, off);
        if (threadIdx.x == 0) chunk_entries[c] = e;
    }
}

// One workgroup per segment: chunk_sums become the exclusive sums over the
// segment's chunks before (DIRECT, short segments: the hist rows
// become the exclusive sums over the blocks before, and no k_bin_chunks runs); lists[segment][super-tile] the start of each list
// within the segment (one past the last: the segment's kept entries);
// seg_entries the segment's emitted entries (the capacity's measure).
template <bool DIRECT>
__global__ void __launch_bounds__(1024) k_bin_top(uint32_t* __restrict__ hist,
                                                  const unsigned long long* __restrict__ partials,
                                                  uint2* __restrict__ chunk_sums, int words, SegLayout sg,
                                                  const unsigned long long* __restrict__ chunk_entries,
                                                  uint32_t* __restrict__ lists,
                                                  unsigned long long* __restrict__ seg_entries) {
    __shared__ uint32_t s_w[16];
    const int nba = ceil_div(sg.la, kBinBlock), nbb = ceil_div(sg.lb, kBinBlock);
    const int nca = ceil_div(nba, kBinChunk), ncb = ceil_div(nbb, kBinChunk);
    const int s = (int)blockIdx.x, tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int c0 = s < sg.na ? s * nca : sg.na * nca + (s - sg.na) * ncb;
    const int nc = s < sg.na ? nca : ncb;
    const int b0 = s < sg.na ? s * nba : sg.na * nba + (s - sg.na) * nbb, nb = s < sg.na ? nba : nbb;
    uint2 run = make_uint2(0u, 0u);
    if (DIRECT && tid < words) {
        uint32_t* col = hist + (size_t)b0 * words + tid;
        uint32_t sum = 0u;  // two 16-bit counts
        for (int k = 0; k < nb; k += 8) {  // eight loads in flight
            uint32_t v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = k + q < nb ? col[(size_t)(k + q) * words] : 0u;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (k + q < nb) {
                    col[(size_t)(k + q) * words] = sum;
                    sum += v[q];
                }
        }
        run = make_uint2(sum & 0xFFFFu, sum >> 16);
    }
    if (!DIRECT && tid < words) {
        uint2* col = chunk_sums + (size_t)c0 * words + tid;
        int k = 0;
        for (; k + 8 <= nc; k += 8) {  // eight loads in flight
            uint2 v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = col[(size_t)(k + q) * words];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                col[(size_t)(k + q) * words] = run;
                run.x += v[q].x;
                run.y += v[q].y;
            }
        }
        for (; k < nc; ++k) {
            const uint2 v = col[(size_t)k * words];
            col[(size_t)k * words] = run;
            run.x += v.x;
            run.y += v.y;
        }
    }
    const uint32_t sum = run.x + run.y;
    uint32_t incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) s_w[w] = incl;
    __syncthreads();
    uint32_t start = incl - sum;
    for (int q = 0; q < w; ++q) start += s_w[q];
    lists += (size_t)s * (2 * words + 1);
    if (tid < words) {
        lists[2 * tid] = start;
        lists[2 * tid + 1] = start + run.x;
        if (tid == words - 1) lists[2 * words] = start + sum;
    }
    if (tid < 64) {
        unsigned long long e = 0ull;
        if (DIRECT) e = tid < nb ? partials[b0 + tid] : 0ull;
        else
            for (int k = tid; k < nc; k += 64) e += chunk_entries[c0 + k];
        for (int off = 32; off > 0; off >>= 1) e += (unsigned long long)__shfl_xor((long long)e, off);
        if (tid == 0) seg_entries[s] = e;
    }
}

// Writes the pass's entries (super-tile relative to the view's grid | tile
// mask << 16, splat id) to entries[cbase[v0] ..), the segments one after
// another, their super-tiles' lists in order, and the lists' ranges.  The
// capacity check is coarse_finalize's, on the emitted entries.  Workgroups map
// to blocks (bin_order) so that one XCD's (every eighth) take kBinRun
// consecutive blocks, whose runs of a super-tile's list adjoin: their lines
// fill in one L2.
// (every other round of 8 kBinRun blocks gives the XCDs their runs in reverse:
// nearer splats, which come first, have more entries)
constexpr int kBinRun = 64;
__device__ __forceinline__ int bin_order(int i, int n) {
    const int round = i / (8 * kBinRun), k = i - round * (8 * kBinRun);
    if ((round + 1) * (8 * kBinRun) > n) return i;
    const int xcd = (round & 1) ? 7 - (k & 7) : k & 7;
    return round * (8 * kBinRun) + xcd * kBinRun + (k >> 3);
}
// NT: 512 threads share a block's 256 splats where the grid's bits leave room
// for few blocks per CU (scatter_threads), else 256.
template <int TILE, int NT>
__global__ void __launch_bounds__(NT) k_bin_scatter(
    const uint32_t* __restrict__ sorted_gid, SegLayout sg, int n_seg, const uint64_t* __restrict__ rect_sorted,
    const CullShape* __restrict__ shapes, const uint2* __restrict__ spans, const ViewParams* __restrict__ views,
    int v0, int v1, const uint32_t* __restrict__ hist, int words, const uint2* __restrict__ chunk_sums,
    const uint32_t* __restrict__ lists, const unsigned long long* __restrict__ seg_entries, uint64_t ccap,
    unsigned long long* cbase, Status* status, unsigned long long* eff_count, uint2* __restrict__ entries,
    int64_t* __restrict__ ranges) {
    constexpr uint32_t S = (uint32_t)super_factor(TILE);
    constexpr int kBinWaveSplats = kBinBlock * 64 / NT;
    constexpr int kBinHeld = NT == 256 ? 4 : 3;  // items per lane kept in registers between marking and writing
    __shared__ uint32_t s_pre[256];
    __shared__ uint64_t s_rect[256];
    __shared__ uint32_t s_gid[256];
    __shared__ uint32_t s_rows[kBinBlock / kBinWaveSplats];  // rows of super-tiles of each wave's splats
    extern __shared__ __align__(16) uint32_t s_dyn[];  // start of the block's run per super-tile, then its bits
    const int tid = (int)threadIdx.x, lane = __lane_id(), w = tid >> 6;
    const unsigned long long base = cbase[v0];
    // the segments' kept entries before this one, and the pass's emitted ones
    unsigned long long C = lane < n_seg ? seg_entries[lane] : 0ull;
    const uint32_t kept = lane < n_seg ? lists[(size_t)lane * (2 * words + 1) + 2 * words] : 0u;
    for (int off = 32; off > 0; off >>= 1) C += (unsigned long long)__shfl_xor((long long)C, off);
    if (blockIdx.x == 0 && tid == 0) coarse_finalize(C, ccap, (int)S, cbase, v0, v1, status, eff_count);
    if (base + C > ccap) return;  // uniform: no list (the ranges stay empty)
    const BinBlock bb = bin_block(bin_order((int)blockIdx.x, (int)gridDim.x), sg, views, v0);
    unsigned long long before = lane < bb.seg ? (unsigned long long)kept : 0ull;
    for (int off = 32; off > 0; off >>= 1) before += (unsigned long long)__shfl_xor((long long)before, off);
    const unsigned long long first = base + before;  // of the segment
    const uint32_t* l = lists + (size_t)bb.seg * (2 * words + 1);
    if (bb.block == 0)
        for (int t = tid; t < bb.supers; t += NT) {
            ranges[2 * ((size_t)bb.super_base + t)] = (int64_t)(first + l[t]);
            ranges[2 * ((size_t)bb.super_base + t) + 1] = (int64_t)(first + l[t + 1]);
        }
    uint32_t* s_run = s_dyn;
    uint32_t* s_bits = s_dyn + 2 * words;
    constexpr int BW = kBinBlock / 32;  // words of bits per super-tile
    {
        const int nba = ceil_div(sg.la, kBinBlock), nbb = ceil_div(sg.lb, kBinBlock);
        const int nca = ceil_div(nba, kBinChunk), ncb = ceil_div(nbb, kBinChunk);
        const int chunk = (bb.seg < sg.na ? bb.seg * nca : sg.na * nca + (bb.seg - sg.na) * ncb) + bb.block / kBinChunk;
        const int b = bb.block + (bb.seg < sg.na ? bb.seg * nba : sg.na * nba + (bb.seg - sg.na) * nbb);
        for (int k = tid; k < words; k += NT) {
            const uint32_t h = hist[(size_t)b * words + k];
            const uint2 cs = chunk_sums ? chunk_sums[(size_t)chunk * words + k] : make_uint2(0u, 0u);
            s_run[2 * k] = l[2 * k] + cs.x + (h & 0xFFFFu);
            s_run[2 * k + 1] = l[2 * k + 1] + cs.y + (h >> 16);
        }
        for (int k = tid; k < bb.supers * BW; k += NT) s_bits[k] = 0u;
    }
    static_assert(NT >= kBinBlock && kBinWaveSplats * (NT / 64) == kBinBlock, "");
    if (tid < kBinBlock) {  // (whole waves)
        const int j = bb.j0 + tid;
        uint64_t rect = kRectNone;
        if (tid < bb.n) {
            rect = rect_sorted[j];
            s_gid[tid] = sorted_gid[j];
        }
        const uint32_t rows = bin_rows<TILE>(rect);
        uint32_t incl = rows;
        for (int off = 1; off < kBinWaveSplats; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off, kBinWaveSplats);
            if ((lane & (kBinWaveSplats - 1)) >= off) incl += y;
        }
        s_pre[tid] = incl - rows;
        s_rect[tid] = rect;
        if ((tid & (kBinWaveSplats - 1)) == kBinWaveSplats - 1) s_rows[tid / kBinWaveSplats] = incl;
    }
    __syncthreads();
    const uint32_t total = s_rows[w];
    const int w0 = w * kBinWaveSplats;
    // an item's spans (from the table, or found again) and columns
    const auto load = [&](uint32_t p, BinItem& it, uint32_t e[S], uint32_t& c0, uint32_t& c1) {
        it = bin_item<TILE, kBinWaveSplats>(p, s_pre + w0, s_rect + w0);
        const size_t jj = (size_t)bb.j0 + w0 + it.g;
        if (it.flags == 0ull) {
            const uint2 b = spans[jj * kBinSlots + it.slot];
            const uint32_t x[4] = {b.x & 0xFFFFu, b.x >> 16, b.y & 0xFFFFu, b.y >> 16};
#pragma unroll
            for (uint32_t q = 0; q < S; ++q)
                e[q] = x[q] != 0u ? (it.tx0 + (x[q] & 0xFFu)) | ((it.tx0 + (x[q] >> 8)) << 16) : 0u;
        } else {
            item_spans<TILE>(it, it.flags == kRectFull ? nullptr : &shapes[jj], e);
        }
        item_columns<TILE>(e, c0, c1);
    };
    const auto mark = [&](const BinItem& it, uint32_t c0, uint32_t c1) {
        if (c0 > c1) return;
        const uint32_t g = (uint32_t)(w0 + it.g), at = it.row * (uint32_t)bb.sx;
        for (uint32_t t = at + c0 / S; t <= at + c1 / S; ++t) atomicOr(&s_bits[t * BW + (g >> 5)], 1u << (g & 31u));
    };
    BinItem it[kBinHeld];
    uint32_t e[kBinHeld][S], c0[kBinHeld], c1[kBinHeld];
#pragma unroll
    for (int q = 0; q < kBinHeld; ++q)
        if ((uint32_t)(q * 64 + lane) < total) load((uint32_t)(q * 64 + lane), it[q], e[q], c0[q], c1[q]);
#pragma unroll
    for (int q = 0; q < kBinHeld; ++q)
        if ((uint32_t)(q * 64 + lane) < total) mark(it[q], c0[q], c1[q]);
    for (uint32_t p = (uint32_t)(kBinHeld * 64 + lane); p < total; p += 64) {
        BinItem i;
        uint32_t ee[S], a, b;
        load(p, i, ee, a, b);
        mark(i, a, b);
    }
    __syncthreads();
    uint2* out = entries + first;
    const uint32_t seg_kept = l[2 * words];
    const auto put = [&](const BinItem& it, const uint32_t e[S], uint32_t c0, uint32_t c1) {
        const uint32_t g = (uint32_t)(w0 + it.g), at = it.row * (uint32_t)bb.sx, id = s_gid[g];
        // the bits below the splat's own, word by word
        uint32_t below[BW];
#pragma unroll
        for (int q = 0; q < BW; ++q)
            below[q] = (uint32_t)q < (g >> 5) ? 0xFFFFFFFFu : ((uint32_t)q == (g >> 5) ? (1u << (g & 31u)) - 1u : 0u);
        if (c0 > c1) return;
        // each tile row's kept columns as bits from a super-tile column on, 32
        // of them at a time
        uint32_t r[S];
        for (uint32_t sc = c0 / S, left = 0u; sc <= c1 / S; ++sc, --left) {
            if (left == 0u) {
                left = 32u / S;
                const uint32_t x0 = sc * S;
#pragma unroll
                for (uint32_t q = 0; q < S; ++q) {
                    const uint32_t lo = max(e[q] & 0xFFFFu, x0), hi = min(e[q] >> 16, x0 + 32u);
                    r[q] = lo < hi ? (0xFFFFFFFFu >> (32u - (hi - lo))) << (lo - x0) : 0u;
                }
            }
            const uint32_t t = at + sc;
            uint32_t m = 0u;
#pragma unroll
            for (uint32_t q = 0; q < S; ++q) {
                m |= (r[q] & ((1u << S) - 1u)) << (q * S);
                r[q] >>= S;
            }
            const uint4* bits = reinterpret_cast<const uint4*>(s_bits + t * BW);
            const uint4 lo = bits[0], hi = bits[1];
            const uint32_t rank = (uint32_t)(__popc(lo.x & below[0]) + __popc(lo.y & below[1]) + __popc(lo.z & below[2]) +
                                             __popc(lo.w & below[3]) + __popc(hi.x & below[4]) + __popc(hi.y & below[5]) +
                                             __popc(hi.z & below[6]) + __popc(hi.w & below[7]));
            const uint32_t pos = s_run[t] + rank;
            if (pos < seg_kept) out[pos] = make_uint2(t | (m << 16), id);  // (always so: counted alike)
        }
    };
#pragma unroll
    for (int q = 0; q < kBinHeld; ++q)
        if ((uint32_t)(q * 64 + lane) < total) put(it[q], e[q], c0[q], c1[q]);
    for (uint32_t p = (uint32_t)(kBinHeld * 64 + lane); p < total; p += 64) {
        BinItem i;
        uint32_t ee[S], a, b;
        load(p, i, ee, a, b);
        put(i, ee, a, b);
    }
}

__global__ void __launch_bounds__(256) k_ranges(const uint2* __restrict__ entries, uint32_t key_mask,
                                                const unsigned long long* eff_count,
                                                const unsigned long long* base_ptr, int64_t* __restrict__ ranges) {
    const uint64_t n = *eff_count;
    const int64_t base = base_ptr ? (int64_t)*base_ptr : 0;
    entries += base;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t t = entries[i].x & key_mask;
        if (i == 0 || (entries[i - 1].x & key_mask) != t) ranges[2 * (size_t)t] = base + (int64_t)i;
        if (i + 1 == n || (entries[i + 1].x & key_mask) != t) ranges[2 * (size_t)t + 1] = base + (int64_t)i + 1;
    }
}

__global__ void k_fill_u64(unsigned long long* p, size_t n, unsigned long long val) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = val;
}
// Backward: workgroup k < passes.n (order_blocks = passes.n) orders pass k
// from the forward's per-bucket tile counts (an exclusive scan, then one
// scatter pass over the tiles; ties in any order), or, with order_blocks = 0,
// the order comes from a sort (k_bwd_order_keys); the other workgroups zero g2
// when a backward has used it since the forward (*dirty) or when force is set.
// Counts that do not add up to the pass's tiles give the identity order.
__global__ void __launch_bounds__(1024) k_bwd_prologue(float* __restrict__ g2, size_t n_g2,
                                                       const unsigned long long* __restrict__ dirty, int force,
                                                       const uint32_t* __restrict__ tcost,
                                                       const uint32_t* __restrict__ thist, PassTiles passes,
                                                       int order_blocks, uint32_t* __restrict__ order) {
    const int k = (int)blockIdx.x;
    if (k < order_blocks) {
        __shared__ uint32_t s_pos[kCostBuckets];
        __shared__ uint32_t s_total, s_bad;
        static_assert(kCostBuckets == 16 * 64, "one wave scans the buckets");
        const int tid = threadIdx.x, nt = blockDim.x;
        const int t0 = passes.tile0[k], n = passes.tile0[k + 1] - t0;
        const uint32_t* h = thist + (size_t)k * kCostBuckets;
        order += t0;
        if (tid < 64) {
            uint32_t v[16], sum = 0u;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                v[i] = h[16 * tid + i];
                sum += v[i];
            }
            uint32_t incl = sum;
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t y = (uint32_t)__shfl_up((int)incl, off);
                if (tid >= off) incl += y;
            }
            uint32_t run = incl - sum;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                s_pos[16 * tid + i] = run;
                run += v[i];
            }
            if (tid == 63) s_total = run;
        }
        if (tid == 0) s_bad = 0u;
        __syncthreads();
        if (s_total == (uint32_t)n) {
            for (int t = tid; t < n; t += nt) {
                const uint32_t pos = atomicAdd(&s_pos[cost_bucket(tcost[t0 + t])], 1u);
                if (pos < (uint32_t)n) order[pos] = (uint32_t)t;
                else s_bad = 1u;
            }
        }
        __syncthreads();
        if (s_total != (uint32_t)n || s_bad)
            for (int t = tid; t < n; t += nt) order[t] = (uint32_t)t;
        return;
    }
    if (!force && *dirty == 0ull) return;  // the records are as the forward left them (uniform)
    const size_t nb = (size_t)(gridDim.x - order_blocks);
    const size_t i0 = (size_t)(k - order_blocks) * blockDim.x + threadIdx.x, step = nb * blockDim.x;
    if ((reinterpret_cast<uintptr_t>(g2) & 15u) == 0 && (n_g2 & 3) == 0) {  // 16-byte stores
        float4* g4 = reinterpret_cast<float4*>(g2);
        for (size_t i = i0; i < n_g2 / 4; i += step) g4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        for (size_t i = i0; i < n_g2; i += step) g2[i] = 0.0f;
    }
}

// Sort keys of the backward's tile order when a pass has too many tiles for one
// workgroup: per global tile t of pass k, key (k, cost bucket), value t - tile0[k].
__global__ void __launch_bounds__(256) k_bwd_order_keys(const uint32_t* __restrict__ tcost, PassTiles passes,
                                                        uint32_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    const int t = blockIdx.x * 256 + (int)threadIdx.x;
    if (t >= passes.tile0[passes.n]) return;
    int k = 0;
    while (k + 1 < passes.n && passes.tile0[k + 1] <= t) ++k;
    keys[t] = ((uint32_t)k << 10) | cost_bucket(tcost[t]);
    vals[t] = (uint32_t)(t - passes.tile0[k]);
}

__global__ void k_fill_f32(float* p, size_t n, float val) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = val;
}

int coarse_count_blocks(int n) { return ceil_div(n, 256); }
void launch_coarse_count(const uint32_t* sorted_gid, int n, int N, SegLayout sg, const Rec* recs,
                         const ViewParams* views, int v0, int tile, int S, uint32_t* cnt, uint64_t* rect_sorted,
                         CullShape* shapes, uint32_t* spans, unsigned long long* partials, hipStream_t st) {
    if (n == 0) return;
    const int nb = coarse_count_blocks(n);
#define H4D_COARSE_COUNT(T) \
    k_coarse_count<T><<<nb, 256, 0, st>>>(sorted_gid, n, N, sg, recs, views, v0, cnt, rect_sorted, shapes, spans, partials)
    if (tile == 8) H4D_COARSE_COUNT(8);
    else if (tile == 16) H4D_COARSE_COUNT(16);
    else H4D_COARSE_COUNT(32);
#undef H4D_COARSE_COUNT
}

BinPlan bin_plan(const SegLayout& sg, int n_groups, int max_supers) {
    BinPlan p;
    const int64_t nba = ceil_div(sg.la, kBinBlock), nbb = ceil_div(sg.lb, kBinBlock);
    p.n_seg = sg.na + n_groups;
    p.blocks = sg.na * nba + n_groups * nbb;
    p.chunks = sg.na * ceil_div((int)nba, kBinChunk) + n_groups * (int64_t)ceil_div((int)nbb, kBinChunk);
    p.direct = nba <= kBinDirect && nbb <= kBinDirect;
    p.words = (max_supers + 3) / 4 * 2;  // (even: the bits behind the runs' starts stay 16-byte aligned)
    auto take = [&](size_t bytes) {
        const size_t o = p.bytes;
        p.bytes = (p.bytes + bytes + 255) / 256 * 256;
        return o;
    };
    p.hist = take(4 * (size_t)p.blocks * p.words);
    p.partials = take(8 * (size_t)p.blocks);
    p.chunk_sums = take(8 * (size_t)p.chunks * p.words);
    p.chunk_entries = take(8 * (size_t)p.chunks);
    p.lists = take(4 * (size_t)p.n_seg * (2 * p.words + 1));
    p.seg_entries = take(8 * (size_t)p.n_seg);
    return p;
}

// Dynamic LDS of the scatter above which a CU holds so few of its workgroups
// that twice the threads per block pay (2704 x 2028 views, 50 KB: 0.123 ->
// 0.101 ms for 1M splats; 1352 x 1014 ones, 13 KB: 0.0176 -> 0.020 ms for 250k).
constexpr size_t kBinWideLds = 32 * 1024;
void launch_bin_ranked(const BinPlan& p, void* work, const uint32_t* sorted_gid, int N, SegLayout sg, const Rec* recs,
                       const ViewParams* views, int v0, int v1, int tile, uint64_t* rect_sorted, CullShape* shapes,
                       uint32_t* spans, uint64_t ccap, unsigned long long* cbase, Status* status,
                       unsigned long long* eff_count, uint2* entries, int64_t* ranges, hipStream_t st) {
    char* w = static_cast<char*>(work);
    uint32_t* hist = reinterpret_cast<uint32_t*>(w + p.hist);
    unsigned long long* partials = reinterpret_cast<unsigned long long*>(w + p.partials);
    uint2* chunk_sums = reinterpret_cast<uint2*>(w + p.chunk_sums);
    unsigned long long* chunk_entries = reinterpret_cast<unsigned long long*>(w + p.chunk_entries);
    uint32_t* lists = reinterpret_cast<uint32_t*>(w + p.lists);
    unsigned long long* seg_entries = reinterpret_cast<unsigned long long*>(w + p.seg_entries);
    const int nb = (int)p.blocks, words = p.words;
    uint2* table = reinterpret_cast<uint2*>(spans);
    const size_t count_lds = 4 * (size_t)words;
    const size_t scatter_lds = 4 * (size_t)(2 * words) * (1 + kBinBlock / 32);
#define H4D_BIN_SCATTER(T, NT)                                                                                         \
    k_bin_scatter<T, NT><<<nb, NT, scatter_lds, st>>>(sorted_gid, sg, p.n_seg, rect_sorted, shapes, table, views, v0,  \
                                                      v1, hist, words, chunk_sums, lists, seg_entries, ccap, cbase,    \
                                                      status, eff_count, entries, ranges)
#define H4D_BIN(T)                                                                                                     \
    do {                                                                                                               \
        k_bin_count<T><<<nb, 256, count_lds, st>>>(sorted_gid, N, sg, recs, views, v0, rect_sorted, shapes, table,     \
                                                   partials, hist, words);                                             \
        if (p.direct) {                                                                                                \
            chunk_sums = nullptr;                                                                                      \
            k_bin_top<true><<<p.n_seg, 1024, 0, st>>>(hist, partials, nullptr, words, sg, nullptr, lists, seg_entries); \
        } else {                                                                                                       \
            k_bin_chunks<<<(unsigned)(p.chunks * ceil_div(words, 64)), 256, 0, st>>>(hist, words, sg, partials,        \
                                                                                     chunk_sums, chunk_entries);       \
            k_bin_top<false><<<p.n_seg, 1024, 0, st>>>(nullptr, nullptr, chunk_sums, words, sg, chunk_entries, lists,  \
                                                       seg_entries);                                                   \
        }                                                                                                              \
        if (scatter_lds > kBinWideLds) H4D_BIN_SCATTER(T, 512);                                                        \
        else H4D_BIN_SCATTER(T, 256);                                                                                  \
    } while (0)
    if (tile == 8) H4D_BIN(8);
    else if (tile == 16) H4D_BIN(16);
    else H4D_BIN(32);
#undef H4D_BIN
#undef H4D_BIN_SCATTER
}
void launch_coarse_offsets(const uint32_t* cnt, int n, unsigned long long* partials, uint64_t ccap, int S,
                           unsigned long long* cbase, int v0, int v1, Status* status, unsigned long long* eff_count,
                           unsigned long long* offsets, uint32_t* run_start, uint64_t run_cap, hipStream_t st) {
    const int nb = coarse_count_blocks(n);
    if (n > 0 && nb <= kDirectParts) {
        k_coarse_down_direct<<<nb, 256, 0, st>>>(cnt, n, partials, nb, ccap, S, cbase, v0, v1, status, eff_count,
                                                 offsets, run_start, run_cap);
        return;
    }
    k_coarse_top<<<1, 1024, 0, st>>>(partials, nb, ccap, S, cbase, v0, v1, status, eff_count);
    if (n > 0) k_coarse_down<<<nb, 256, 0, st>>>(cnt, n, partials, nb, offsets, run_start, run_cap);
}
void launch_coarse_emit(const unsigned long long* offsets, const uint32_t* run_start, int n, SegLayout sg,
                        const uint64_t* rect_sorted, const CullShape* shapes, const uint32_t* spans,
                        const ViewParams* views, int v0, int tile, int S, uint64_t capacity,
                        const unsigned long long* eff_count, uint32_t* keys, uint32_t* vals, hipStream_t st) {
    if (n == 0 || capacity == 0) return;
    // (32 views of 1M Gaussians in one pass: about 25 runs of 256 entries per workgroup)
    const int nb = (int)std::min<uint64_t>(65536, (capacity + 255) / 256);
#define H4D_COARSE_EMIT(T) \
    k_coarse_emit<T><<<nb, 256, 0, st>>>(offsets, run_start, n, sg, rect_sorted, shapes, spans, views, v0, eff_count, \
                                         keys, vals)
    if (tile == 8) H4D_COARSE_EMIT(8);
    else if (tile == 16) H4D_COARSE_EMIT(16);
    else H4D_COARSE_EMIT(32);
#undef H4D_COARSE_EMIT
}
void launch_ranges(const uint2* entries, uint32_t key_mask, const unsigned long long* eff_count,
                   const unsigned long long* base, int64_t* ranges, hipStream_t st) {
    k_ranges<<<2048, 256, 0, st>>>(entries, key_mask, eff_count, base, ranges);
}
bool launch_bwd_prologue(float* g2, size_t n_g2, const unsigned long long* dirty, int force, const uint32_t* tcost,
                         const uint32_t* thist, const PassTiles& passes, const OrderSort& sort, uint32_t* order,
                         hipStream_t st) {
    int most = 0;
    for (int k = 0; k < passes.n; ++k) most = std::max(most, passes.tile0[k + 1] - passes.tile0[k]);
    const bool by_sort = most > kOrderBlockTiles;
    // a grid-stride loop of 16-byte stores over at most 4096 workgroups (which
    // return at once when nothing is to be cleared)
    const int fill = (int)std::max<size_t>(1, std::min<size_t>(4096, (n_g2 + 4095) / 4096));
    const int ob = by_sort ? 0 : passes.n;
    k_bwd_prologue<<<ob + fill, 1024, 0, st>>>(g2, n_g2, dirty, force, tcost, thist, passes, ob, order);
    if (!by_sort) return true;
    // one stable sort of (pass, cost bucket) keys over all tiles: every pass's
    // tiles in a run of their own, by decreasing cost
    const int tiles = passes.tile0[passes.n];
    k_bwd_order_keys<<<(tiles + 255) / 256, 256, 0, st>>>(tcost, passes, sort.keys, sort.vals);
    int bits = 10;
    while ((1 << (bits - 10)) < passes.n) ++bits;
    const int np = (bits + kMaxRadixBits - 1) / kMaxRadixBits;
    uint32_t *kin = sort.keys, *vin = sort.vals, *kalt = sort.keys2, *valt = sort.vals2;
    for (int p = 0, shift = 0; p < np; ++p) {
        const int nb = (bits - shift + (np - p) - 1) / (np - p);
        uint32_t* vout = p == np - 1 ? order : valt;
        if (!launch_radix_pass(kin, vin, kalt, vout, nullptr, (uint64_t)tiles, (uint64_t)tiles, shift, nb, sort.hist,
                               sort.hist_words, sort.totals, sort.totals_words, nullptr, st))
            return false;
        std::swap(kin, kalt);
        vin = vout;
        valt = (vout == sort.vals2) ? sort.vals : sort.vals2;
        shift += nb;
    }
    return true;
}

void launch_fill_u64(unsigned long long* p, size_t n, unsigned long long val, hipStream_t st) {
    if (n == 0) return;
    const int nb = (int)std::min<size_t>(4096, (n + 255) / 256);
    k_fill_u64<<<nb, 256, 0, st>>>(p, n, val);
}
// (n <= 64; dst may be pinned host memory)
__global__ void k_copy_words(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst, int n) {
    if ((int)threadIdx.x < n) dst[threadIdx.x] = src[threadIdx.x];
}
hipError_t launch_copy_words(const uint32_t* src, uint32_t* dst, int n, hipStream_t st) {
    if (n < 0 || n > 64) return hipErrorInvalidValue;
    void* args[] = {&src, &dst, &n};
    return hipLaunchKernel((const void*)k_copy_words, dim3(1), dim3(64), args, 0, st);
}

void launch_fill_f32(float* p, size_t n, float val, hipStream_t st) {
    if (n == 0) return;
    const int nb = (int)std::min<size_t>(8192, (n + 255) / 256);
    k_fill_f32<<<nb, 256, 0, st>>>(p, n, val);
}

}  // namespace h4d
