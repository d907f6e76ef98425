// Stable least-significant-digit radix sort of (uint64 key, int32 value) pairs, 8-bit
// digits, one pass per digit.  Each pass:
//   histogram  per tile of 2048 items the digit counts in LDS, stored
//   scatter    each item's destination: where its tile's items of the digit start, plus
//              the items of that digit before it in the tile.  A wavefront takes 512
//              consecutive items, all loaded at once, and counts them per digit in its own
//              row of LDS as it ranks them 64 at a time (the lanes with the same digit
//              found by ballots), so that it waits for no other; the wavefronts' rows are
//              summed once.
// Up to kDirectTiles tiles the scatter finds its tile's starts itself, each thread adding
// one digit's counts over the tiles; beyond, an exclusive scan of the counts (stored digit
// by digit) does so in three more launches.  (Five launches a pass and a barrier for every
// 256 items took 37 us a pass on 262,144 items and 33 on 8,000; this takes 18 and 10.)
// Equal keys keep their input order, so the sort is stable.
#include "common.hpp"
#include "rhs_common.hpp"

namespace sph {
namespace {

constexpr int kDigitBits = 8;
constexpr int kDigits = 1 << kDigitBits;
constexpr int kRounds = 8;  // items of a thread
constexpr int kSortTile = kBlock * kRounds;
constexpr int kWaves = kBlock / 64;
constexpr int64_t kDirectTiles = 256;

__device__ inline int digit_of(uint64_t key, int shift) { return (int)((key >> shift) & (kDigits - 1)); }

// Where digit d's count of a tile stands.
template <bool kDirect>
__device__ inline int64_t hist_at(int d, int64_t tile, int64_t tiles) {
    return kDirect ? tile * kDigits + d : d * tiles + tile;
}

template <bool kDirect>
__global__ __launch_bounds__(kBlock) void k_digit_hist(const uint64_t *__restrict__ key, int64_t n,
                                                       int shift, int32_t *__restrict__ hist,
                                                       int64_t tiles) {
    __shared__ int32_t cnt[kDigits];
    cnt[threadIdx.x] = 0;  // kBlock == kDigits
    const int64_t base = (int64_t)blockIdx.x * kSortTile + threadIdx.x;
    uint64_t k[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) k[r] = base + r * kBlock < n ? key[base + r * kBlock] : 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (base + r * kBlock < n) atomicAdd(&cnt[digit_of(k[r], shift)], 1);
    __syncthreads();
    hist[hist_at<kDirect>(threadIdx.x, blockIdx.x, tiles)] = cnt[threadIdx.x];
}

template <bool kDirect>
__global__ __launch_bounds__(kBlock) void k_digit_scatter(const uint64_t *__restrict__ kin,
                                                          const int32_t *__restrict__ vin,
                                                          int64_t n, int shift,
                                                          const int32_t *__restrict__ hist,
                                                          int64_t tiles,
                                                          uint64_t *__restrict__ kout,
                                                          int32_t *__restrict__ vout) {
    __shared__ int32_t cnt[kWaves][kDigits];  // a wavefront's items per digit, then their places
    __shared__ int32_t part[kWaves];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;  // lanes below this one
    const int64_t base = (int64_t)blockIdx.x * kSortTile + w * (64 * kRounds) + lane;
    uint64_t k[kRounds];
    int32_t v[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const bool valid = base + 64 * r < n;
        k[r] = valid ? kin[base + 64 * r] : 0;
        v[r] = valid ? vin[base + 64 * r] : 0;
    }
    // digit t: its items in all tiles, and in the tiles before this one
    int all = 0, start = 0;
    if constexpr (kDirect) {
#pragma unroll 8
        for (int64_t i = 0; i < tiles; ++i) {
            const int c = hist[hist_at<true>(t, i, tiles)];
            all += c;
            start += i < blockIdx.x ? c : 0;
        }
    } else {
        start = hist[hist_at<false>(t, blockIdx.x, tiles)];  // (scanned)
    }
#pragma unroll
    for (int q = 0; q < kWaves; ++q) cnt[q][t] = 0;
    __syncthreads();
    int rank[kRounds];  // among the wavefront's items of the digit
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const bool valid = base + 64 * r < n;
        const int d = digit_of(k[r], shift);
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kDigitBits; ++b) {
            const uint64_t ones = __ballot((d >> b) & 1);
            same &= ((d >> b) & 1) ? ones : ~ones;
        }
        const int below = __popcll(same & lt), before = cnt[w][d];
        rank[r] = before + below;
        wave_sync();
        if (valid && below == 0) cnt[w][d] = before + __popcll(same);  // the digit's lowest lane
        wave_sync();
    }
    if constexpr (kDirect) {  // the digits before this one
        int incl = all;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(incl, o);
            if (lane >= o) incl += u;
        }
        if (lane == 63) part[w] = incl;
        start += incl - all;
    }
    __syncthreads();
    if constexpr (kDirect)
        for (int q = 0; q < w; ++q) start += part[q];
#pragma unroll
    for (int q = 0; q < kWaves; ++q) {
        const int c = cnt[q][t];
        cnt[q][t] = start;
        start += c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (base + 64 * r < n) {
            const int dst = cnt[w][digit_of(k[r], shift)] + rank[r];
            kout[dst] = k[r];
            vout[dst] = v[r];
        }
}

}  // namespace

// Scratch elements (int32) of radix_sort_pairs for n items.
size_t radix_sort_tmp_elems(int64_t n) {
    const int64_t tiles = (n + kSortTile - 1) / kSortTile;
    const int64_t m = tiles * kDigits;
    return (size_t)(m + 1) + scan_tmp_elems(m + 1) + 64;
}

// Sorts (key[0], val[0]) by bits [0, bits) of the keys; the result is in buffer
// *which (0 or 1) of the double buffers.  tmp: radix_sort_tmp_elems(n) int32.
int radix_sort_pairs(uint64_t *key[2], int32_t *val[2], int64_t n, int bits, int32_t *tmp,
                     int *which, hipStream_t s) {
    *which = 0;
    if (n <= 1) return SPH_OK;
    if (n >= ((int64_t)1 << 31)) return fail(SPH_ERR_INVALID_ARG, "radix sort of 2^31 items or more");
    const int64_t tiles = (n + kSortTile - 1) / kSortTile;
    const int64_t m = tiles * kDigits;
    int32_t *hist = tmp;
    int32_t *scan = tmp + m + 1;
    int cur = 0;
    for (int shift = 0; shift < bits; shift += kDigitBits) {
        if (tiles <= kDirectTiles) {
            k_digit_hist<true><<<(unsigned)tiles, kBlock, 0, s>>>(key[cur], n, shift, hist, tiles);
            SPH_LAUNCHED();
            k_digit_scatter<true><<<(unsigned)tiles, kBlock, 0, s>>>(
                key[cur], val[cur], n, shift, hist, tiles, key[cur ^ 1], val[cur ^ 1]);
            SPH_LAUNCHED();
        } else {
            k_digit_hist<false><<<(unsigned)tiles, kBlock, 0, s>>>(key[cur], n, shift, hist, tiles);
            SPH_LAUNCHED();
            int rc = exclusive_scan_i32(hist, hist, m, scan, s);
            if (rc) return rc;
            k_digit_scatter<false><<<(unsigned)tiles, kBlock, 0, s>>>(
                key[cur], val[cur], n, shift, hist, tiles, key[cur ^ 1], val[cur ^ 1]);
            SPH_LAUNCHED();
        }
        cur ^= 1;
    }
    *which = cur;
    return SPH_OK;
}

}  // namespace sph
