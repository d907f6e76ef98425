// Frozen candidate-pair list ("interactionsList" of section 3.5.2 with a
// skin): for every slot, the slots whose distance was below h + skin when the
// list was built.  While every particle stays within skin/2 of its position at
// build time this is a superset of its partners, and the pair kernels re-test
// d^2 < h^2 exactly at the current positions.
//
// Layout: slots are grouped in blocks of 64 (one wavefront); inside block B the
// j-th candidate of the block's lane l sits at slot[block_start[B] + 64 j + l],
// so the j-th loads of a wavefront are contiguous.  Each block's lists are padded to
// its longest, whose length (the largest count of its 64 slots) is the block's number
// of steps.  A block's room, 64 times the largest bound of its slots (the slots of the
// cells within reach of each slot, counted without a distance test), is fixed before
// the one pass that tests and writes the candidates, so no count pass is needed.
#include "common.hpp"
#include "rhs_common.hpp"
#include "sweep.hpp"
#include "window.hpp"

namespace sph {
namespace {

constexpr int kWave = 64;

// Gathers the positions into slot order and bounds every slot's candidates: the slots of
// the cells within reach of its position (each candidate lies in one of them, within delta
// of its cell's box), self included.  sizes[B] = 64 * (largest bound of block B).  (The
// gather, the bounds and the blocks' largest in three passes took 35 us on 30,000
// particles and 133 on a million; this takes 21 and 110.)
__global__ __launch_bounds__(kBlock) void k_pl_bound(GridDev g, const double *__restrict__ x,
                                                     const double *__restrict__ y,
                                                     const double *__restrict__ z, int64_t n,
                                                     double reach, double *__restrict__ x0,
                                                     int64_t *__restrict__ sizes,
                                                     int32_t *__restrict__ status) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int b = 0;
    if (s < n) {
        const int a = g.perm[s];
        const double px = x[a], py = y[a], pz = z[a];
        if (!within_cell(g, (int)s, px, py, pz)) raise_flag(status, SPH_ERR_STALE_GRID);
        x0[3 * s + 0] = px;
        x0[3 * s + 1] = py;
        x0[3 * s + 2] = pz;
        for_each_row(g, px, py, pz, reach, [&](int s0, int s1) { b += s1 - s0; });
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) b = max(b, __shfl_xor(b, o));
    if (__lane_id() == 0 && s < n) sizes[s / kWave] = (int64_t)kWave * b;
}

// Fill pass, one wavefront per group of 64 slots.  The fill writes entry j of lane l
// at block_start[B] + 64 j + l, pads every list to the group's longest with the slot
// itself (n - 1 for the lanes past n), so every entry of a group's steps is a valid
// slot and readers of whole groups load without guards, and writes each slot's count
// (and its partners at the grid's h).
//
// A compact group sweeps, once and cooperatively, the cell rows of its bounding box
// widened by the reach, from the middle of the region outwards (z, then y), x
// increasing along a row and slots increasing inside a cell; each list holds its
// slot's candidates in that order.  The sweep goes in passes of up to 64 rows: each
// lane takes one row (culled against the group's box as a whole) and lays the row's
// runs of consecutive slots out in LDS, in row order; the pass's candidates are then
// streamed 64 at a time, so that the loads of a pass do not wait on one another row by
// row.  Each loaded candidate is culled, one lane per candidate, against the group's
// box widened by the radius (one farther away is no lane's candidate); the survivors
// are packed in order into an LDS buffer, which the 64 lanes test against their own
// slots 64 candidates at a time (broadcast reads).  A group spread over a region of
// more than kSpread times one slot's cells sweeps tile by tile, or per lane, in the order
// of for_each_row either way.

__global__ __launch_bounds__(kBlock) void k_pl_fill(GridDev g, const double *__restrict__ x0,
                                                    int64_t n, double r2, double reach,
                                                    int32_t *__restrict__ count,
                                                    const int64_t *__restrict__ block_start,
                                                    int32_t *__restrict__ slot, double h2,
                                                    int32_t *__restrict__ partners) {
    __shared__ double lds[kBlock / 64][3][2 * kWave];
    __shared__ int32_t lds_t[kBlock / 64][2 * kWave];
    __shared__ int32_t lds_r[kBlock / 64][2][kRunCap];
    double(*cand)[2 * kWave] = lds[threadIdx.x >> 6];
    int32_t *cand_t = lds_t[threadIdx.x >> 6];
    int32_t *run_s0 = lds_r[threadIdx.x >> 6][0];   // a run's first slot (first its cell)
    int32_t *run_pre = lds_r[threadIdx.x >> 6][1];  // candidates before it in the pass
    const int lane = __lane_id();
    const int64_t nb = (n + kWave - 1) / kWave;
    // (neighbouring groups on one XCD: a million particles 715 us in launch order, 660 so)
    const int64_t B = xcd_block(gridDim.x) * (kBlock / kWave) + (threadIdx.x >> 6);
    if (B >= nb) return;  // whole wavefront past the end
    const int64_t s = B * kWave + lane;
    const bool act = s < n;
    const int64_t sa = act ? s : B * kWave;  // lanes past n stand on the group's first slot
    const double xa = x0[3 * sa], ya = x0[3 * sa + 1], za = x0[3 * sa + 2];
    const int64_t base = block_start[B] + lane;
    const int64_t room = (block_start[B + 1] - block_start[B]) / kWave;
    int c = 0, np = 0;  // candidates and partners (d^2 < h^2) among them
    int32_t *const group = slot + block_start[B];  // entry j of lane l at group[64 j + l]
    const int iroom = (int)min(room, (int64_t)(INT_MAX >> 6));
    auto hit = [&](int t, double d) {
        // the bound pass gave room for every candidate; the guard keeps a write
        // inside the group even so
        if (c < iroom) group[(uint32_t)((c << 6) + lane)] = t;
        np += d < h2;
        ++c;
    };
    GroupParts parts(g, act, sa, xa, ya, za, reach);
    while (parts.todo) {
        bool single;
        const bool in = parts.next(g, act, xa, ya, za, reach, single);
        const GroupBox &box = parts.box;
        if (single) {
            if (in)
                for_each_row(g, xa, ya, za, reach, [&](int s0, int s1) {
                    for (int t = s0; t < s1; ++t) {
                        if (t == s) continue;
                        const double d = dist2_exact(xa, ya, za, x0[3 * t], x0[3 * t + 1], x0[3 * t + 2]);
                        if (d < r2) hit(t, d);
                    }
                });
            continue;
        }
        // the cull keeps every candidate within the radius of a point of the box, with a
        // margin far above the rounding of either distance
        const double rb2 = r2 * (1.0 + 1e-6);
        int pend = 0;  // candidates waiting in the buffer (wavefront-uniform)
        auto test = [&](int m) {
            int k = 0;
            for (; k + 4 <= m; k += 4) {  // four distances, then their hits
                int t[4];
                double d[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    t[q] = cand_t[k + q];
                    d[q] = dist2_exact(xa, ya, za, cand[0][k + q], cand[1][k + q], cand[2][k + q]);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (in && d[q] < r2 && t[q] != (int)s) hit(t[q], d[q]);
            }
            for (; k < m; ++k) {
                const int t = cand_t[k];
                const double d = dist2_exact(xa, ya, za, cand[0][k], cand[1][k], cand[2][k]);
                if (in && d < r2 && t != (int)s) hit(t, d);
            }
        };
        // one candidate per lane (t, where valid): loaded, culled, packed behind the
        // waiting ones; 64 waiting are tested
        auto push = [&](bool valid, int t) {
            bool keep = false;
            double px = 0.0, py = 0.0, pz = 0.0;
            if (valid) {
                px = x0[3 * (int64_t)t];
                py = x0[3 * (int64_t)t + 1];
                pz = x0[3 * (int64_t)t + 2];
                keep = box.dist2(px, py, pz) < rb2;
            }
            const unsigned long long mk = __ballot(keep);
            if (keep) {
                const int at = pend + (int)__builtin_amdgcn_mbcnt_hi(
                                          (unsigned)(mk >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mk, 0));
                cand[0][at] = px;
                cand[1][at] = py;
                cand[2][at] = pz;
                cand_t[at] = t;
            }
            pend += __popcll(mk);
            wave_sync();
            if (pend >= kWave) {
                test(kWave);
                pend -= kWave;
                wave_sync();
                if (lane < pend) {  // the rest to the front (reads above kWave only)
                    cand[0][lane] = cand[0][kWave + lane];
                    cand[1][lane] = cand[1][kWave + lane];
                    cand[2][lane] = cand[2][kWave + lane];
                    cand_t[lane] = cand_t[kWave + lane];
                }
                wave_sync();
            }
        };
        const int nrows = box.rows();
        for (int rb = 0, skip = 0; rb < nrows;) {
            const RunPass p = lay_runs(g, box, parts.tiles == 0, reach, rb, skip, run_s0, run_pre);
            // the pass's candidates in order, 64 at a time
            for (int f0 = 0; f0 < p.total; f0 += kWave)
                push(f0 + lane < p.total, slot_of_run(f0 + lane, p.runs, run_s0, run_pre));
            wave_sync();
        }
        test(pend);
        wave_sync();
    }
    // the group's steps: its longest list (at most its room)
    int steps = min((int64_t)c, room);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) steps = max(steps, __shfl_xor(steps, o));
    const int32_t pad = act ? (int32_t)s : (int32_t)(n - 1);
    for (int64_t j = c; j < steps; ++j) slot[base + kWave * j] = pad;
    if (act) {
        count[s] = c;
        if (partners) partners[s] = np;
    }
}

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
// meets the candidates, took three times the fill's own time.  This takes 83 us, and 3.8 ms
// on an 8,388,608-particle non-uniform set, where it moves 13 GB.)
constexpr int kPageTable = 512;
constexpr int kMaxPages = 384;       // the table stays open
constexpr int kMaxLocals = 2047;     // locals numbered
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
            // (fewer pages than places are entered: a free place is met)
            while (__ballot(open[0] || open[1] || open[2] || open[3])) {
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

size_t pairs_ws_bytes(int64_t n) {
    Carve c(nullptr);
    const int64_t nb = (n + kWave - 1) / kWave;
    c.take<int64_t>(nb);
    c.take<int64_t>(scan_tmp_elems(nb));
    return c.used;
}

}  // namespace sph

using namespace sph;

extern "C" int sph_build_pairs(sph_grid *grid, const double *x, const double *y, const double *z,
                               sph_pairs *out, int32_t *count, int32_t *partners,
                               int64_t *block_start, int32_t *slot, int64_t capacity, double *x0,
                               int64_t *needed, void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    int rc = check_grid(grid);
    if (rc) return rc;
    if (!x || !y || !z || !out || !count || !block_start || !x0 || !needed || !ws ||
        (!slot && capacity > 0))
        return fail(SPH_ERR_INVALID_ARG, "null pointer");
    const int64_t n = grid->n;
    const size_t need = pairs_ws_bytes(n);
    if (ws_bytes < need) return fail(SPH_ERR_WORKSPACE, "workspace %zu < %zu bytes", ws_bytes, need);
    hipStream_t s = (hipStream_t)stream;
    Carve c(ws);
    const int64_t nb = (n + 63) / 64;
    int64_t *sizes = c.take<int64_t>(nb);
    int64_t *tmp = c.take<int64_t>(scan_tmp_elems(nb));
    GridDev g = grid_dev(grid);
    g.pl_count = nullptr;  // the cells, not a previous list, locate the candidates
    g.pl_block = nullptr;
    g.pl_slot = nullptr;
    g.pl_x0 = nullptr;
    const double radius = grid->h + grid->skin;
    const double r2 = radius * radius * (1.0 + 1e-12);
    const double reach = (radius + g.delta) * (1.0 + 1e-9);
    if ((rc = clear_status(ws, s))) return rc;
    const double h2 = grid->h * grid->h;  // the partner test of sph_neighbours at grid->h
    k_pl_bound<<<blocks_for(n), kBlock, 0, s>>>(g, x, y, z, n, reach, x0, sizes, c.status());
    SPH_LAUNCHED();
    if ((rc = exclusive_scan_i64(sizes, block_start, nb, tmp, s))) return rc;
    int64_t total = 0;
    int32_t flag = 0;
    SPH_HIP_TRY(hipMemcpyAsync(&total, block_start + nb, sizeof total, hipMemcpyDeviceToHost, s));
    SPH_HIP_TRY(hipMemcpyAsync(&flag, c.status(), sizeof flag, hipMemcpyDeviceToHost, s));
    SPH_HIP_TRY(hipStreamSynchronize(s));
    *needed = total;
    if (flag) return fail(flag, "device flag %d raised while building the pair list", flag);
    if (total > capacity)
        return fail(SPH_ERR_CAPACITY, "pair list needs %lld entries, capacity %lld",
                    (long long)total, (long long)capacity);
    k_pl_fill<<<blocks_for(nb, kBlock / 64), kBlock, 0, s>>>(g, x0, n, r2, reach, count,
                                                              block_start, slot, h2, partners);
    SPH_LAUNCHED();
    if (grid->skin > 0.0) {  // (the kernels that read the hints are chosen by the skin too)
        k_pl_hints<<<blocks_for(nb, kBlock / kWave), kBlock, 0, s>>>(n, count, block_start, slot);
        SPH_LAUNCHED();
    }
    out->n = n;
    out->radius = radius;
    out->skin = grid->skin;
    out->count = count;
    out->block_start = block_start;
    out->slot = slot;
    out->capacity = capacity;
    out->x0 = x0;
    out->partners = partners;
    grid->pairs = out;
    return SPH_OK;
}
