// Sweeps of the cells around a group of 64 slots: which rows of cells the bounding box of
// the group or of a part of it, widened by the reach, meets, and the runs of consecutive
// slots these rows hold.
#pragma once

#include "common.hpp"
#include "rhs_common.hpp"

namespace sph {

// A region of more than kSpread times the cells of one slot's is not worth one sweep.  A
// group's is mostly so where the group runs on from the end of one tile of cells to the
// start of the next: one in about fourteen on a lattice with 14 particles a cell.  Such a
// group is swept tile by tile while its slots lie in at most kMaxTiles tiles, slot by slot
// (each lane by itself) otherwise, in sparse parts of a set.  (The right-hand side from the
// cells of 200,000 particles in two spheres: 916 us with all such groups slot by slot, 502
// with at most 4 tiles, 374 with 8 and with 64.)
constexpr double kSpread = 8.0;
constexpr int kMaxTiles = 8;
constexpr int kRunCap = 256;  // runs of one pass (LDS)

// Distance from the interval [b0, b1] to the slab of cell i along one axis (the
// first and last cells extend to infinity, as in slab_gap).
__device__ inline double box_gap(double b0, double b1, double lo, double cell, int i, int ncell) {
    const double a = lo + cell * i;
    const double b = a + cell;
    double g = 0.0;
    if (i > 0 && b1 < a) g = a - b1;
    if (i < ncell - 1 && b0 > b) g = b0 - b;
    return g;
}

__device__ inline double wave_min(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}

__device__ inline double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}

struct GroupBox {
    double x0, x1, y0, y1, z0, z1;     // box of the 64 positions
    int ix0, ix1, iy0, iy1, iz0, iz1;  // cells within reach of it
    bool spread;

    __device__ int rows() const { return (iz1 - iz0 + 1) * (iy1 - iy0 + 1); }
    // squared distance of a point from the box
    __device__ double dist2(double px, double py, double pz) const {
        const double ex = fmax(fmax(x0 - px, px - x1), 0.0);
        const double ey = fmax(fmax(y0 - py, py - y1), 0.0);
        const double ez = fmax(fmax(z0 - pz, pz - z1), 0.0);
        return ex * ex + ey * ey + ez * ez;
    }
};

// (in: the lanes whose positions count)
__device__ inline GroupBox group_box(const GridDev &g, bool in, double xa, double ya, double za,
                                     double reach) {
    constexpr double far = 1.7976931348623157e308;
    GroupBox b;
    b.x0 = wave_min(in ? xa : far), b.x1 = wave_max(in ? xa : -far);
    b.y0 = wave_min(in ? ya : far), b.y1 = wave_max(in ? ya : -far);
    b.z0 = wave_min(in ? za : far), b.z1 = wave_max(in ? za : -far);
    b.iz0 = cell_index(b.z0 - reach, g.loz, g.inv_cell, g.nz);
    b.iz1 = cell_index(b.z1 + reach, g.loz, g.inv_cell, g.nz);
    b.iy0 = cell_index(b.y0 - reach, g.loy, g.inv_cell, g.ny);
    b.iy1 = cell_index(b.y1 + reach, g.loy, g.inv_cell, g.ny);
    b.ix0 = cell_index(b.x0 - reach, g.lox, g.inv_cell, g.nx);
    b.ix1 = cell_index(b.x1 + reach, g.lox, g.inv_cell, g.nx);
    const double own = 2.0 * reach * g.inv_cell + 1.0;  // cells along one axis of one slot
    const double cells = (double)(b.ix1 - b.ix0 + 1) * (b.iy1 - b.iy0 + 1) * (b.iz1 - b.iz0 + 1);
    b.spread = cells > kSpread * own * own * own;
    return b;
}

// The parts a group is swept in: next() gives the lanes of the next part and its box until
// todo is empty.
struct GroupParts {
    GroupBox box;
    int tile, tiles;  // this lane's tile of cells; the group's tiles, 0: swept as a whole
    unsigned long long todo;

    __device__ GroupParts(const GridDev &g, bool act, int64_t s, double xa, double ya, double za,
                          double reach)
        : box(group_box(g, act, xa, ya, za, reach)), tile(0), tiles(0), todo(__ballot(act)) {
        if (!box.spread) return;
        tile = g.cell_of[s] >> 6;  // (64 cells a tile)
        for (unsigned long long m = todo; m && tiles <= kMaxTiles; ++tiles)
            m &= ~__ballot(act && tile == first_tile(m));
    }
    __device__ int first_tile(unsigned long long m) const {
        return __builtin_amdgcn_readlane(tile, __ffsll((long long)m) - 1);
    }
    // true for this lane if it belongs to the part; single: the part goes slot by slot
    __device__ bool next(const GridDev &g, bool act, double xa, double ya, double za, double reach,
                         bool &single) {
        const bool in = act && (tiles == 0 || tiles > kMaxTiles || tile == first_tile(todo));
        todo &= ~__ballot(in);
        if (tiles > 0 && tiles <= kMaxTiles) box = group_box(g, in, xa, ya, za, reach);
        single = box.spread;
        return in;
    }
};

// One pass of a sweep: the rows from row rb of a region on that fit it, or, where row rb
// alone has more than kRunCap runs, that many of its runs from run skip on; rb and skip
// are advanced.  runs runs of consecutive slots (run j: slots from s0[j] on, pre[j]
// candidates before it), `total` candidates in all.  A whole group's rows go from the
// middle of the region outwards (z, then y): its lanes then meet their partners at more
// even rates, so that the rows of the list they fill together are completed sooner.  A
// part's rows go in increasing z and y, the order of for_each_row.
struct RunPass {
    int runs, total;
};

// (by one whole wavefront; s0, pre: kRunCap words of LDS each)
__device__ inline RunPass lay_runs(const GridDev &g, const GroupBox &b, bool whole, double reach,
                                   int &rb, int &skip, int32_t *run_s0, int32_t *run_pre) {
    const int lane = __lane_id();
    const double rr = reach * reach;
    const int nyr = b.iy1 - b.iy0 + 1, nrows = b.rows();
    auto middle_out = [](int r, int lo, int hi) {  // r-th of c, c - 1, c + 1, c - 2, ...
        const int c = (lo + hi) >> 1, a = c - lo;
        return r <= 2 * a ? c + ((r & 1) ? -((r + 1) >> 1) : (r >> 1)) : hi;
    };
    RunPass p;
    // this lane's row of the pass: its cells in x and its number of runs
    const int r = rb + lane;
    int iy = 0, iz = 0, xr0 = 0, xr1 = -1, nr = 0;
    if (r < nrows) {
        iz = whole ? middle_out(r / nyr, b.iz0, b.iz1) : b.iz0 + r / nyr;
        iy = whole ? middle_out(r % nyr, b.iy0, b.iy1) : b.iy0 + r % nyr;
        const double gz = box_gap(b.z0, b.z1, g.loz, g.cell, iz, g.nz);
        const double gy = box_gap(b.y0, b.y1, g.loy, g.cell, iy, g.ny);
        const double d2 = gz * gz + gy * gy;
        if (gz * gz < rr && d2 < rr) {
            const double w = sqrt(rr - d2) * (1.0 + 1e-9);
            xr0 = cell_index(b.x0 - w, g.lox, g.inv_cell, g.nx);
            xr1 = cell_index(b.x1 + w, g.lox, g.inv_cell, g.nx);
            for_each_cell_run(g, iy, iz, xr0, xr1, [&](int, int) { ++nr; });
        }
    }
    // runs before this lane's (exclusive scan over the lanes)
    int off = nr;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(off, o);
        if (lane >= o) off += v;
    }
    off -= nr;
    // the rows that fit the pass: a prefix of the lanes
    const int rows = __popcll(__ballot(r < nrows && off + nr <= kRunCap));
    if (rows == 0) {
        const int all = __builtin_amdgcn_readfirstlane(nr);
        int j = -skip;
        for_each_cell_run(g, __builtin_amdgcn_readfirstlane(iy), __builtin_amdgcn_readfirstlane(iz),
                          __builtin_amdgcn_readfirstlane(xr0), __builtin_amdgcn_readfirstlane(xr1),
                          [&](int c0, int c1) {
                              if (lane == 0 && j >= 0 && j < kRunCap) {
                                  run_s0[j] = c0;
                                  run_pre[j] = c1;
                              }
                              ++j;
                          });
        p.runs = min(kRunCap, all - skip);
        skip += kRunCap;
        if (skip >= all) {
            skip = 0;
            rb += 1;
        }
    } else {
        p.runs = __shfl(off + nr, rows - 1);
        if (lane < rows && nr > 0) {  // (a culled row has no runs)
            int j = off;
            for_each_cell_run(g, iy, iz, xr0, xr1, [&](int c0, int c1) {
                run_s0[j] = c0;
                run_pre[j] = c1;
                ++j;
            });
        }
        rb += rows;
    }
    wave_sync();
    // the runs' slots: cells to slot ranges, and their lengths scanned
    int len[kRunCap / 64], sum = 0;
#pragma unroll
    for (int q = 0; q < kRunCap / 64; ++q) {
        const int j = kRunCap / 64 * lane + q;
        len[q] = 0;
        if (j < p.runs) {
            const int s0 = g.cell_start[run_s0[j]];
            len[q] = g.cell_start[run_pre[j]] - s0;
            run_s0[j] = s0;
        }
        sum += len[q];
    }
    int before = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(before, o);
        if (lane >= o) before += v;
    }
    p.total = __shfl(before, 63);
    before -= sum;
#pragma unroll
    for (int q = 0; q < kRunCap / 64; ++q) {
        const int j = kRunCap / 64 * lane + q;
        if (j < p.runs) run_pre[j] = before;
        before += len[q];
    }
    wave_sync();
    return p;
}

// Slot of a pass's candidate f (its run: the last with pre <= f); any slot number for f
// past the last.
__device__ inline int slot_of_run(int f, int runs, const int32_t *run_s0, const int32_t *run_pre) {
    int lo = 0, hi = runs;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (run_pre[mid] <= f) lo = mid; else hi = mid;
    }
    return run_s0[lo] + (f - run_pre[lo]);
}

}  // namespace sph
