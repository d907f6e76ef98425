// The kernel that leaves the hints of window.hpp behind the entries of a pair list.
#pragma once

#include "common.hpp"
#include "rhs_common.hpp"
#include "window.hpp"

namespace sph {
namespace {

constexpr int kWave = 64;

// Largest value over the wavefront, in every lane (rows of 16 by shifts, then the rows'
// last lanes broadcast: no LDS round trips).
__device__ inline int wave_max_i32(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));  // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));  // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));  // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));  // row_shr:8
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));  // row_bcast:15
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// The hints behind a group's entries (window.hpp), one wavefront per group.  The slots a
// group names lie in a hundred or so pages of 16 consecutive ones.  A first pass over the
// list enters the pages in a small hash table in LDS (linear probing), numbers them in the
// order of the steps that name them and marks the slots named, a word of bits per page;
// the locals are the marked slots, page by page; a second pass turns the entries' places
// in the table into locals.  What bounds it is the chain of memory and LDS round trips,
// hence sixteen steps' entries loaded together and four probed together.  A wavefront's
// LDS operations keep their order, so a place of the table is taken by a plain write that
// is read back.  (A table of the slots themselves, probed up to a dozen times by some lane
// at every step, took 150 us on 262,144 particles; four wavefronts on one group with
// compare-and-swap 110; pages of 64, whose locals follow the steps less closely, made the
// pair kernels of dense sets slower by a fifth; numbers given by the fill itself, as it
// meets the candidates, took three times the fill's own time.  This takes 85 us on the
// 262,144 particles.)
constexpr int kPageTable = 512;
constexpr int kMaxPages = 384;       // pages of a group with hints: probes stay short
constexpr int kBatch = 4;            // chunks whose entries are loaded together

__global__ __launch_bounds__(kBlock) void k_pl_hints(int64_t n, const int32_t *__restrict__ count,
                                                     const int64_t *__restrict__ block_start,
                                                     int32_t *__restrict__ slot) {
    struct Pages {
        int32_t key[kPageTable];      // page (slot / 16), -1: free
        uint32_t bits[kPageTable];    // its slots named
        uint16_t number[kPageTable];  // its number
        uint16_t base[kPageTable];    // locals of the pages numbered before it
        uint16_t order[kMaxPages + kWave];  // page number -> place
    };
    __shared__ Pages lds[kBlock / kWave];
    Pages &P = lds[threadIdx.x >> 6];
    const int lane = __lane_id();
    const int64_t nb = (n + kWave - 1) / kWave;
    const int64_t B = xcd_block(gridDim.x) * (kBlock / kWave) +
                      __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (B >= nb) return;  // whole wavefront past the end
    const int64_t s = B * kWave + lane;
    const int64_t base = block_start[B], end = block_start[B + 1];
    const int64_t room = (end - base) / kWave;
    const HintLayout h = hint_layout(room, slot);
    if (h.steps <= 0) return;  // no room for a header either
    const int cnt = s < n ? count[s] : 0;
    const int steps = list_steps(cnt);
    if (steps + kHintHeader / 64 > room) return;
    const int32_t *const row = slot + base + lane;
    int32_t *const head = slot + end - kHintHeader;
    int32_t *const uni = head - h.uni;
    uint64_t *const hint = reinterpret_cast<uint64_t *>(uni) + lane;
    if (lane == 0) head[0] = 0;  // no hints until they are all there
    if (steps > h.steps) return;
    const int chunks = (steps + kChunkSteps - 1) / kChunkSteps;
    for (int i = lane; i < kPageTable; i += kWave) {
        P.key[i] = -1;
        P.bits[i] = 0;
    }
    wave_sync();
    int pages = 0;
    for (int c0 = 0; c0 < chunks; c0 += kBatch) {
        int32_t t[kBatch][kChunkSteps];
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
#pragma unroll
            for (int i = 0; i < kChunkSteps; ++i) {
                const int j = kChunkSteps * (c0 + k) + i;
                t[k][i] = j < cnt ? row[(int64_t)64 * j] : -1;
            }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            if (c0 + k >= chunks) break;
            int at[kChunkSteps], pg[kChunkSteps];
            bool open[kChunkSteps], fresh[kChunkSteps];
#pragma unroll
            for (int i = 0; i < kChunkSteps; ++i) {
                pg[i] = t[k][i] >> 4;
                at[i] = (int)((uint32_t)pg[i] * 2654435761u >> 23);  // kPageTable = 2^9 places
                open[i] = t[k][i] >= 0;
                fresh[i] = false;
            }
            bool any_fresh = false;
            // A chunk may bring a page from each of its entries, more than the table has places
            // left.  Each turn takes every open entry one place on, and a place once taken
            // stays taken: an entry that has met all places without its page's or a free
            // one finds the table full, and the group gets no hints.
            for (int turn = 0; __ballot(open[0] || open[1] || open[2] || open[3]); ++turn) {
                if (turn == kPageTable) return;
                int32_t key[kChunkSteps];
#pragma unroll
                for (int i = 0; i < kChunkSteps; ++i) key[i] = P.key[at[i]];
                const bool take = (open[0] && key[0] < 0) || (open[1] && key[1] < 0) ||
                                  (open[2] && key[2] < 0) || (open[3] && key[3] < 0);
                if (__ballot(take)) {
                    any_fresh = true;
                    wave_sync();
#pragma unroll
                    for (int i = 0; i < kChunkSteps; ++i)
                        if (open[i] && key[i] < 0) P.key[at[i]] = pg[i];
                    wave_sync();
#pragma unroll
                    for (int i = 0; i < kChunkSteps; ++i) {
                        const bool was_free = open[i] && key[i] < 0;
                        key[i] = P.key[at[i]];
                        fresh[i] = fresh[i] || (was_free && key[i] == pg[i]);
                    }
                }
#pragma unroll
                for (int i = 0; i < kChunkSteps; ++i) {
                    open[i] = open[i] && key[i] != pg[i];
                    if (open[i]) at[i] = (at[i] + 1) & (kPageTable - 1);
                }
            }
            if (any_fresh) {
                // one of the entries that name a new page numbers it
                wave_sync();
#pragma unroll
                for (int i = kChunkSteps - 1; i >= 0; --i)
                    if (fresh[i]) P.number[at[i]] = (uint16_t)(kChunkSteps * lane + i);
                wave_sync();
                uint16_t who[kChunkSteps];
#pragma unroll
                for (int i = 0; i < kChunkSteps; ++i) who[i] = P.number[at[i]];
                wave_sync();
#pragma unroll
                for (int i = 0; i < kChunkSteps; ++i) {
                    fresh[i] = fresh[i] && who[i] == (uint16_t)(kChunkSteps * lane + i);
                    const unsigned long long m = __ballot(fresh[i]);
                    const int p = pages + __popcll(m & ((1ull << lane) - 1));
                    if (fresh[i] && p < kMaxPages) P.order[p] = (uint16_t)at[i];
                    pages += __popcll(m);
                }
                if (pages > kMaxPages) return;  // a set too scattered
            }
            // mark the entries' slots
            uint32_t w[kChunkSteps];
            uint64_t four = 0;
#pragma unroll
            for (int i = 0; i < kChunkSteps; ++i) w[i] = P.bits[at[i]];
#pragma unroll
            for (int i = 0; i < kChunkSteps; ++i) {
                const int b = t[k][i] & 15;
                if (t[k][i] >= 0 && !(w[i] >> b & 1)) atomicOr(&P.bits[at[i]], 1u << b);
                four |= (uint64_t)(uint16_t)(at[i] << 4 | b) << 16 * i;
            }
            hint[-64 * (c0 + k + 1)] = four;  // place of the page and slot of it, for now
        }
    }
    static_assert(kPageTable << 4 <= 0x10000, "a place and a slot of the page fit 16 bits");
    wave_sync();
    // the locals: the marked slots of the pages in turn
    int used = 0;
    for (int p0 = 0; p0 < pages; p0 += kWave) {
        const int p = p0 + lane, at = p < pages ? P.order[p] : 0;
        const uint32_t m = p < pages ? P.bits[at] : 0;
        int sum = __popc(m);
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int v = __shfl_up(sum, o);
            if (lane >= o) sum += v;
        }
        const int first = used + sum - __popc(m);
        used += __builtin_amdgcn_readlane(sum, 63);
        if (used > min(h.uni, kMaxLocals)) return;  // too many
        if (p < pages) P.base[at] = (uint16_t)first;
        const int page = p < pages ? P.key[at] : 0;
        int l = first;
#pragma unroll
        for (int b = 0; b < 16; ++b)
            if (m >> b & 1) uni[l++] = 16 * page + b;
    }
    wave_sync();
    wait_vm();
    int least = 0xffff, most = 0;   // of the round at hand
    int my_lo = 0xffff, my_hi = 0;  // lane r: round r's
    for (int c0 = 0; c0 < chunks; c0 += kBatch) {
        uint64_t e[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) e[k] = c0 + k < chunks ? hint[-64 * (c0 + k + 1)] : 0;
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int c = c0 + k;
            if (c >= chunks) break;
            uint64_t four = 0;
#pragma unroll
            for (int i = 0; i < kChunkSteps; ++i) {
                const int x = (int)(e[k] >> 16 * i) & 0xffff, at = x >> 4 & (kPageTable - 1);
                const int l = P.base[at] + __popc(P.bits[at] & ((1u << (x & 15)) - 1));
                if (kChunkSteps * c + i < cnt) {
                    least = min(least, l);
                    most = max(most, l + 1);
                    four |= (uint64_t)l << 16 * i;
                }
            }
            hint[-64 * (c + 1)] = four;
            if ((c + 1) * kChunkSteps % kRoundSteps == 0 || c + 1 == chunks) {
                const int lo = 0xffff - wave_max_i32(0xffff - least), hi = wave_max_i32(most);
                if (lane == c * kChunkSteps / kRoundSteps) {
                    my_lo = lo;
                    my_hi = hi;
                }
                least = 0xffff;
                most = 0;
            }
        }
    }
    // a round's lowest counts those after it, its highest those before it
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int lo = __shfl_down(my_lo, o), hi = __shfl_up(my_hi, o);
        if (lane + o < kWave) my_lo = min(my_lo, lo);
        if (lane >= o) my_hi = max(my_hi, hi);
    }
    head[64 + lane] = (int)((uint32_t)my_hi << 16 | (uint32_t)my_lo);
    if (lane < 3) head[lane] = lane == 0 ? kHintMagic : lane == 1 ? used : steps;
}

}  // namespace
}  // namespace sph
