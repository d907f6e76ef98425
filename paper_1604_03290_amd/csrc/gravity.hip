// Barnes-Hut self-gravity with monopoles (section 3.3, eq. gravitational_force)
// on the octree of section 3.5.1.
//
// Instead of inserting particles under locks into a pointer octree, the tree is
// read off the Morton order of the particles: with 63-bit keys interleaving the
// 21-bit integer coordinates (x bit first in each triple), the cube of depth d
// holding a particle is its key's 3d-bit prefix, and the inner nodes (cubes with
// two or more particles) are the runs of equal prefixes of length >= 2 in the
// sorted keys.  Laid out in depth-first pre-order (children in octant order, the
// same order as the keys), the tree needs no child pointers: an item is followed
// by its first child, and each item stores `skip`, the first item after its
// subtree.  A node starting at sorted position i spans up to the first position
// whose key leaves its prefix (a binary search); the nodes starting at i are the
// depths D_{i-1} < d <= D_i, D_i being the depth shared by keys i and i + 1.
//
//   keys      bounding cube (reduction), integer coordinates, keys
//   sort      the library's stable LSD radix sort of (key, user index), 8 passes of
//             8 bits (sort.hip)
//   depth     D_i and the number of nodes starting at i; scan -> item offsets
//   items     leaves (position, mass) and inner nodes (depth, skip), and the list of
//             inner nodes (the k-th inner node in pre-order is list[k])
//   monopole  one pass per depth, deepest first, over the inner-node list: mass and
//             centre of mass of each node of that depth over its children in octant
//             order
//   walk      one wavefront walks the tree for its 64 particles together, 64 nodes at a
//             time (k_walk); every particle takes exactly the terms of its own walk
#include "common.hpp"
#include "rhs_common.hpp"
#include "sweep.hpp"
#include "timing.hpp"

namespace sph {
namespace {

// One 48-byte tree item:
// pm = (x, y, z, m): a leaf's position and mass, an inner node's centre of mass and
// mass once the monopole pass ran; link = (skip, info), info = depth for an inner node
// and -1 - i for the leaf of sorted position i.
struct __attribute__((aligned(16))) Item {
    double4 pm;
    int2 link;
    int2 pad;
};

constexpr int kDepthMax = 21;  // 3 x 21 key bits

// ------------------------------------------------------------------ keys --
__global__ __launch_bounds__(kBlock) void k_bbox_partial(const double *__restrict__ x,
                                                         const double *__restrict__ y,
                                                         const double *__restrict__ z, int64_t n,
                                                         double *__restrict__ part) {
    __shared__ double lds[6][kBlock];
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    double v[6];
    if (i < n) {
        v[0] = v[3] = x[i];
        v[1] = v[4] = y[i];
        v[2] = v[5] = z[i];
    } else {
        const int64_t j = (int64_t)blockIdx.x * kBlock;  // first of the block, < n
        v[0] = v[3] = x[j];
        v[1] = v[4] = y[j];
        v[2] = v[5] = z[j];
    }
    for (int c = 0; c < 6; ++c) lds[c][threadIdx.x] = v[c];
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            for (int c = 0; c < 3; ++c)
                lds[c][threadIdx.x] = fmin(lds[c][threadIdx.x], lds[c][threadIdx.x + w]);
            for (int c = 3; c < 6; ++c)
                lds[c][threadIdx.x] = fmax(lds[c][threadIdx.x], lds[c][threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x < 6) part[(int64_t)blockIdx.x * 6 + threadIdx.x] = lds[threadIdx.x][0];
}

// box = (lo x, lo y, lo z, s0)
__global__ __launch_bounds__(kBlock) void k_bbox_final(const double *__restrict__ part,
                                                       int64_t nb, double *__restrict__ box) {
    __shared__ double lds[6][kBlock];
    double v[6];
    for (int c = 0; c < 6; ++c) v[c] = part[c];
    for (int64_t b = threadIdx.x; b < nb; b += kBlock)
        for (int c = 0; c < 6; ++c) {
            const double u = part[b * 6 + c];
            v[c] = c < 3 ? fmin(v[c], u) : fmax(v[c], u);
        }
    for (int c = 0; c < 6; ++c) lds[c][threadIdx.x] = v[c];
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            for (int c = 0; c < 3; ++c)
                lds[c][threadIdx.x] = fmin(lds[c][threadIdx.x], lds[c][threadIdx.x + w]);
            for (int c = 3; c < 6; ++c)
                lds[c][threadIdx.x] = fmax(lds[c][threadIdx.x], lds[c][threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double s0 = 0.0;
        for (int c = 0; c < 3; ++c) {
            const double e = lds[c + 3][0] - lds[c][0];
            if (e > s0) s0 = e;
        }
        box[0] = lds[0][0];
        box[1] = lds[1][0];
        box[2] = lds[2][0];
        box[3] = s0;
    }
}

__device__ inline uint32_t quantise(double v, double lo, double s0) {
    if (!(s0 > 0.0)) return 0u;
    const double u = floor((v - lo) / s0 * 2097152.0);  // 2^21
    if (!(u >= 0.0)) return 0u;  // a non-finite position (flagged by the caller)
    return u >= 2097152.0 ? 2097151u : (uint32_t)u;
}

// spreads the 21 low bits of v to every third bit
__device__ inline uint64_t spread3(uint32_t v) {
    uint64_t x = v & 0x1fffffu;
    x = (x | x << 32) & 0x1f00000000ffffull;
    x = (x | x << 16) & 0x1f0000ff0000ffull;
    x = (x | x << 8) & 0x100f00f00f00f00full;
    x = (x | x << 4) & 0x10c30c30c30c30c3ull;
    x = (x | x << 2) & 0x1249249249249249ull;
    return x;
}

__global__ __launch_bounds__(kBlock) void k_keys(const double *__restrict__ x,
                                                 const double *__restrict__ y,
                                                 const double *__restrict__ z,
                                                 const double *__restrict__ m, int64_t n,
                                                 const double *__restrict__ box,
                                                 uint64_t *__restrict__ key,
                                                 int32_t *__restrict__ idx,
                                                 int32_t *__restrict__ status) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double xi = x[i], yi = y[i], zi = z[i], mi = m[i];
    if (!isfinite(xi) || !isfinite(yi) || !isfinite(zi) || !(mi > 0.0) || !isfinite(mi))
        raise_flag(status, SPH_ERR_DOMAIN);
    const double s0 = box[3];
    const uint32_t qx = quantise(xi, box[0], s0), qy = quantise(yi, box[1], s0),
                   qz = quantise(zi, box[2], s0);
    key[i] = spread3(qx) << 2 | spread3(qy) << 1 | spread3(qz);
    idx[i] = (int32_t)i;
}

// ----------------------------------------------------------------- depth --
// depth shared by sorted keys i and i + 1 (-1 past the last); the number of inner
// nodes that start at i, c_i = max(0, D_i - D_{i-1}), and the deepest node's depth.
__device__ inline int shared_depth(const uint64_t *key, int64_t i, int64_t n) {
    if (i < 0) return -1;
    if (i + 1 >= n) return -1;
    const uint64_t d = key[i] ^ key[i + 1];
    const int bits = d ? __clzll((long long)d) - 1 : 63;  // common prefix of the 63-bit keys
    return bits / 3;
}

__global__ __launch_bounds__(kBlock) void k_depth(const uint64_t *__restrict__ key, int64_t n,
                                                  int64_t *__restrict__ cnt,
                                                  int32_t *__restrict__ max_depth) {
    __shared__ int bmax;
    if (threadIdx.x == 0) bmax = -1;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) {
        const int d1 = shared_depth(key, i, n), d0 = shared_depth(key, i - 1, n);
        cnt[i] = d1 > d0 ? d1 - d0 : 0;
        if (d1 >= 0) atomicMax(&bmax, d1);
    } else if (i == n) {
        cnt[n] = 0;
    }
    __syncthreads();
    if (threadIdx.x == 0 && bmax >= 0) atomicMax(max_depth, bmax);
}

// ----------------------------------------------------------------- items --
// Items of sorted position i: its inner nodes (depths D_{i-1} + 1 .. D_i), then its leaf.
__global__ __launch_bounds__(kBlock) void k_items(
    const double *__restrict__ x, const double *__restrict__ y, const double *__restrict__ z,
    const double *__restrict__ m, const uint64_t *__restrict__ key, const int32_t *__restrict__ idx,
    const int64_t *__restrict__ off, int64_t n, int32_t *__restrict__ list,
    Item *__restrict__ it) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int d1 = shared_depth(key, i, n), d0 = shared_depth(key, i - 1, n);
    const int64_t first = i + off[i];
    int64_t t = first;
    const uint64_t ki = key[i];
    for (int d = d0 + 1; d <= d1; ++d, ++t) {
        const int shift = 63 - 3 * d;
        const uint64_t pre = ki >> shift;
        int64_t lo = i + 1, hi = n;  // first position whose prefix differs
        while (lo < hi) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            if ((key[mid] >> shift) == pre)
                lo = mid + 1;
            else
                hi = mid;
        }
        it[t].link = make_int2((int)(lo + off[lo]), d);
        it[t].pm = make_double4(0.0, 0.0, 0.0, 0.0);
        list[off[i] + (t - first)] = (int32_t)t;
    }
    const int a = idx[i];
    it[t].link = make_int2((int)(t + 1), (int)(-1 - i));
    it[t].pm = make_double4(x[a], y[a], z[a], m[a]);
}

// -------------------------------------------------------------- monopole --
__global__ __launch_bounds__(kBlock) void k_monopole(const int32_t *__restrict__ list, int64_t K,
                                                     int depth, Item *__restrict__ it) {
#pragma clang fp contract(off)
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= K) return;
    const int t = list[j];
    const int2 lt = it[t].link;
    if (lt.y != depth) return;
    const int end = lt.x;
    double M = 0.0, mx = 0.0, my = 0.0, mz = 0.0;
    for (int c = t + 1; c < end; c = it[c].link.x) {
        const double4 p = it[c].pm;
        M = M + p.w;
        mx = mx + p.w * p.x;
        my = my + p.w * p.y;
        mz = mz + p.w * p.z;
    }
    it[t].pm = make_double4(mx / M, my / M, mz / M, M);
}

// ------------------------------------------------------------------ walk --
struct GravConsts {
    double G, th2, eps;  // th2 = theta^2
    int64_t n, T;
};

// a += G m_p (x_p - x_a) / (r + eps)^3 for r2 = r^2 > 0, gm = G m_p
__device__ inline void add_term(const GravConsts &k, double gm, double dx, double dy, double dz,
                                double &ax, double &ay, double &az) {
    const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
    if (r2 == 0.0) return;
    const double ir = rsqrt64(r2);
    double id;
    if (k.eps > 0.0) {
        id = rcp64(fma(r2, ir, k.eps));
    } else {
        id = ir;
    }
    const double f = gm * (id * id * id);
    ax = fma(f, dx, ax);
    ay = fma(f, dy, ay);
    az = fma(f, dz, az);
}

// The opening test s / r < theta is taken as s^2 < theta^2 r^2 with
// r^2 = (dx dx + dy dy) + dz dz rounded as written (no fused operations), the same
// arithmetic as the test's definition in the oracle.
__device__ inline double dist2_plain(double dx, double dy, double dz) {
#pragma clang fp contract(off)
    return dx * dx + dy * dy + dz * dz;
}

__device__ inline bool opens_not(double s, double th2, double r2) {
#pragma clang fp contract(off)
    return s * s < th2 * r2;
}

__device__ inline double read_lane(double v, int l) {
    const int2 w = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(
        double, make_int2(__builtin_amdgcn_readlane(w.x, l), __builtin_amdgcn_readlane(w.y, l)));
}

// One wavefront, or kWaves of them, take 64 consecutive particles of the sorted order.  A
// wavefront's work is a stack of ranges of siblings, each with the lanes that walk it; up
// to 64 ranges are taken off the top at a time, one lane looking at the first node of
// each.  A node that even the nearest point of the lanes' box accepts is a term of all the
// range's lanes, a node that even the farthest opens is opened for all; only the nodes
// between are tested by each lane for itself, one after the other.  Terms are gathered in
// LDS with their lanes and added from there, one after the other, without tests or waits.
// So the loads of 64 nodes are in flight together, and what remains is bound by the terms'
// arithmetic, about 30 instructions each.  (A walk of one node at a time, its pointer
// common to the 64 lanes, spent half its time on the chain of loads and half its
// instructions on the tests: 1631 us on 262,144 particles at theta 0.5; this takes 1434.)
//
// With several wavefronts all begin with the root; once kDeal ranges are on the stack each
// keeps every kWaves-th of them (the terms until then are wavefront 0's), and their sums
// are added in order at the end.  That halves the time of a set too small to fill the chip
// with one wavefront per 64 particles, but the beginning is walked by all and the stacks
// are shorter: all of sph_gravity with four and with one, us, 8,000 particles 390 and 625,
// 100,000 (1,563 groups) 569 and 640, 150,000 (2,344 groups) 1360 and 1189.
//
// The stack: taking m ranges leaves at most 2 m (a range's rest, the node's children), so
// that with m at most 32 less than the places left the 32 stay free; when no more are,
// ranges are taken singly, and the topmost range's subtree needs at most one place for
// each level of the tree.
constexpr int kStack = 320;
constexpr int kStackSpare = 32;
static_assert(kStackSpare > kDepthMax + 2, "a walk of single ranges needs a place per level");
constexpr int kTermBatch = 32;  // terms are added when more than these wait

constexpr int kDeal = 32;
constexpr int kWalkWaves = 4;
constexpr int64_t kFewGroups = 1792;  // groups of 64 up to which kWalkWaves take one

template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) void k_walk(GravConsts k, const double *__restrict__ box,
                                             const int32_t *__restrict__ idx,
                                             const Item *__restrict__ it,
                                             const int64_t *__restrict__ off,
                                             const int64_t *__restrict__ cnt,
                                             double *__restrict__ ax_out,
                                             double *__restrict__ ay_out,
                                             double *__restrict__ az_out,
                                             int32_t *__restrict__ count_out) {
    __shared__ int2 lds_range[kWaves][kStack];            // first node, end
    __shared__ uint64_t lds_who[kWaves][kStack];          // its lanes
    __shared__ double4 lds_term[kWaves][kTermBatch + 64];  // position, G m
    __shared__ uint64_t lds_term_who[kWaves][kTermBatch + 64];
    const int lane = __lane_id();
    const int q = kWaves == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int2 *const range = lds_range[q];
    uint64_t *const who = lds_who[q], *const term_who = lds_term_who[q];
    double4 *const term = lds_term[q];
    const int64_t i0 = xcd_block(gridDim.x) * 64;
    if (i0 >= k.n) return;  // whole workgroup past the end
    const bool live = i0 + lane < k.n;
    const int64_t i = live ? i0 + lane : k.n - 1;
    const double4 me = it[i + off[i] + cnt[i]].pm;
    const double xa = me.x, ya = me.y, za = me.z;
    const double bx0 = wave_min(xa), bx1 = wave_max(xa);
    const double by0 = wave_min(ya), by1 = wave_max(ya);
    const double bz0 = wave_min(za), bz1 = wave_max(za);
    const double s0 = box[3];
    double ax = 0.0, ay = 0.0, az = 0.0;
    int terms = 0, pend = 0;
    auto add_terms = [&] {
        wave_sync();
#pragma unroll 4
        for (int e = 0; e < pend; ++e) {
            const double4 p = term[e];
            const int2 w = __builtin_bit_cast(int2, term_who[e]);
            const uint64_t lanes = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(w.y) << 32 |
                                   (uint32_t)__builtin_amdgcn_readfirstlane(w.x);
            if (__builtin_amdgcn_inverse_ballot_w64(lanes)) {
                add_term(k, p.w, p.x - xa, p.y - ya, p.z - za, ax, ay, az);
                ++terms;
            }
        }
        pend = 0;
        wave_sync();
    };
    auto before = [&](unsigned long long m) { return __popcll(m & ((1ull << lane) - 1)); };
    const unsigned long long all = __ballot(live);
    if (lane == 0) {
        range[0] = make_int2(0, (int)k.T);
        who[0] = all;
    }
    int size = 1;
    bool dealt = kWaves == 1;
    while (size > 0) {
        if (!dealt && size >= kDeal) {  // (fewer than 2 kDeal: a round at most doubles it)
            static_assert(2 * kDeal <= 64 * kWalkWaves, "one range per lane is kept");
            dealt = true;
            const int keep = (size - q + kWaves - 1) / kWaves;
            wave_sync();
            const int from = min(q + kWaves * lane, size - 1);
            const int2 r = range[from];
            const uint64_t w = who[from];
            wave_sync();
            if (lane < keep) {
                range[lane] = r;
                who[lane] = w;
            }
            size = keep;
            if (q != 0) {
                ax = ay = az = 0.0;
                terms = pend = 0;
            }
        }
        const int m = min(min(size, 64), max(kStack - size - kStackSpare, 1));
        wave_sync();
        size -= m;
        const bool valid = lane < m;
        const int2 r = valid ? range[size + lane] : make_int2(0, 0);
        const uint64_t mine = valid ? who[size + lane] : 0;
        wave_sync();
        const Item node = it[r.x];
        const double4 p = node.pm;
        const int skip = node.link.x, info = node.link.y;
        uint64_t take = 0, open = 0;  // the lanes that take the node as a term, that open it
        bool between = false;
        double side = 0.0;
        if (valid && info < 0) {
            const int64_t own = (int64_t)(-1 - info) - i0;  // a particle is no term of itself
            take = own >= 0 && own < 64 ? mine & ~(1ull << own) : mine;
        } else if (valid) {
            const double s = ldexp(s0, -info);
            side = s;
            const double nx = fmax(fmax(bx0 - p.x, p.x - bx1), 0.0), fx = fmax(p.x - bx0, bx1 - p.x);
            const double ny = fmax(fmax(by0 - p.y, p.y - by1), 0.0), fy = fmax(p.y - by0, by1 - p.y);
            const double nz = fmax(fmax(bz0 - p.z, p.z - bz1), 0.0), fz = fmax(p.z - bz0, bz1 - p.z);
            // margins far above the rounding of either side
            const double lo = k.th2 * (nx * nx + ny * ny + nz * nz) * (1.0 - 1e-12);
            const double hi = k.th2 * (fx * fx + fy * fy + fz * fz) * (1.0 + 1e-12);
            if (s * s < lo)
                take = mine;
            else if (s * s >= hi)
                open = mine;
            else
                between = true;
        }
        for (unsigned long long b = __ballot(between); b; b &= b - 1) {
            const int l = __ffsll((long long)b) - 1;
            const double dx = read_lane(p.x, l) - xa, dy = read_lane(p.y, l) - ya,
                         dz = read_lane(p.z, l) - za;
            const unsigned long long yes =
                __ballot(opens_not(read_lane(side, l), k.th2, dist2_plain(dx, dy, dz)));
            if (lane == l) {
                take = mine & yes;
                open = mine & ~yes;
            }
        }
        const unsigned long long tm = __ballot(take != 0);
        if (take != 0) {
            const int at = pend + before(tm);
            term[at] = make_double4(p.x, p.y, p.z, k.G * p.w);
            term_who[at] = take;
        }
        pend += __popcll(tm);
        const bool more = valid && skip < r.y;
        const unsigned long long rm = __ballot(more), om = __ballot(open != 0);
        if (more) {
            const int at = size + before(rm);
            range[at] = make_int2(skip, r.y);
            who[at] = mine;
        }
        size += __popcll(rm);
        if (open != 0) {
            const int at = size + before(om);
            range[at] = make_int2(r.x + 1, skip);
            who[at] = open;
        }
        size += __popcll(om);
        if (pend > kTermBatch) {
            if (dealt || q == 0) add_terms();
            pend = 0;
        }
    }
    if (dealt || q == 0) add_terms();
    if constexpr (kWaves > 1) {
        if (!dealt && q != 0) {
            ax = ay = az = 0.0;
            terms = 0;
        }
        double *sum = reinterpret_cast<double *>(lds_term);
        static_assert(sizeof lds_term >= kWaves * 4 * 64 * 8, "the sums fit");
        __syncthreads();
        sum[(4 * q + 0) * 64 + lane] = ax;
        sum[(4 * q + 1) * 64 + lane] = ay;
        sum[(4 * q + 2) * 64 + lane] = az;
        sum[(4 * q + 3) * 64 + lane] = (double)terms;  // (exact)
        __syncthreads();
        if (q != 0) return;
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            ax += sum[(4 * w + 0) * 64 + lane];
            ay += sum[(4 * w + 1) * 64 + lane];
            az += sum[(4 * w + 2) * 64 + lane];
            terms += (int)sum[(4 * w + 3) * 64 + lane];
        }
    }
    if (!live) return;
    const int a = idx[i];
    ax_out[a] = ax;
    ay_out[a] = ay;
    az_out[a] = az;
    if (count_out) count_out[a] = terms;
}

__global__ void k_set_i32(int32_t *p, int32_t v) {
    if (threadIdx.x == 0) p[0] = v;
}

// ------------------------------------------------------------- workspace --
struct GravWs {
    double *part, *box;
    uint64_t *key[2];
    int32_t *idx[2];
    int64_t *cnt, *off, *scan_tmp;
    int32_t *max_depth;
    int32_t *list;
    Item *it;
    int32_t *sort_tmp;
};

int64_t node_capacity(int64_t n, int64_t cap) { return cap > 0 ? cap : 2 * n; }

GravWs carve_grav(Carve &c, int64_t n, int64_t cap) {
    GravWs w;
    w.part = c.take<double>((size_t)blocks_for(n) * 6);
    w.box = c.take<double>(4);
    for (int b = 0; b < 2; ++b) {
        w.key[b] = c.take<uint64_t>(n);
        w.idx[b] = c.take<int32_t>(n);
    }
    w.cnt = c.take<int64_t>(n + 1);
    w.off = c.take<int64_t>(n + 1);
    w.scan_tmp = c.take<int64_t>(scan_tmp_elems(n + 1));
    w.max_depth = c.take<int32_t>(1);
    w.list = c.take<int32_t>(cap);
    w.it = c.take<Item>(n + cap);
    w.sort_tmp = c.take<int32_t>(radix_sort_tmp_elems(n));
    return w;
}

}  // namespace

size_t gravity_ws_bytes(int64_t n, int64_t cap) {
    Carve c(nullptr);
    carve_grav(c, n, node_capacity(n, cap));
    return c.used;
}

}  // namespace sph

using namespace sph;

extern "C" int sph_gravity(const double *x, const double *y, const double *z, const double *m,
                           int64_t n, double G, double theta, double eps, double *ax, double *ay,
                           double *az, int32_t *count, int64_t node_cap, int64_t *nodes_out,
                           void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    if (!x || !y || !z || !m || !ax || !ay || !az || !ws)
        return fail(SPH_ERR_INVALID_ARG, "null pointer");
    if (n < 1 || n > (int64_t)1 << 26) return fail(SPH_ERR_INVALID_ARG, "n must be in [1, 2^26]");
    if (!std::isfinite(G) || !std::isfinite(theta) || !std::isfinite(eps) || theta < 0.0 ||
        theta >= 1.0 || eps < 0.0)
        return fail(SPH_ERR_INVALID_ARG, "finite G, 0 <= theta < 1 and eps >= 0 required");
    const int64_t cap = node_capacity(n, node_cap);
    if (cap > 22 * n) return fail(SPH_ERR_INVALID_ARG, "node_cap above 22 n");
    const size_t need = gravity_ws_bytes(n, node_cap);
    if (ws_bytes < need) return fail(SPH_ERR_WORKSPACE, "workspace %zu < %zu bytes", ws_bytes, need);
    hipStream_t s = (hipStream_t)stream;
    int rc;
    if ((rc = clear_status(ws, s))) return rc;
    Carve c(ws);
    GravWs w = carve_grav(c, n, cap);
    TimedRegion tr("gravity", s);

    const unsigned nb = blocks_for(n);
    k_bbox_partial<<<nb, kBlock, 0, s>>>(x, y, z, n, w.part);
    SPH_LAUNCHED();
    k_bbox_final<<<1, kBlock, 0, s>>>(w.part, nb, w.box);
    SPH_LAUNCHED();
    k_keys<<<nb, kBlock, 0, s>>>(x, y, z, m, n, w.box, w.key[0], w.idx[0], c.status());
    SPH_LAUNCHED();

    int which = 0;
    if ((rc = radix_sort_pairs(w.key, w.idx, n, 63, w.sort_tmp, &which, s))) return rc;
    const uint64_t *key = w.key[which];
    const int32_t *idx = w.idx[which];

    k_set_i32<<<1, 64, 0, s>>>(w.max_depth, -1);
    SPH_LAUNCHED();
    k_depth<<<blocks_for(n + 1), kBlock, 0, s>>>(key, n, w.cnt, w.max_depth);
    SPH_LAUNCHED();
    if ((rc = exclusive_scan_i64(w.cnt, w.off, n + 1, w.scan_tmp, s))) return rc;

    // the tree's size: inner nodes K = off[n], and the deepest node's depth
    int64_t K = 0;
    int32_t dmax = -1;
    SPH_HIP_TRY(hipMemcpyAsync(&K, w.off + n, sizeof K, hipMemcpyDeviceToHost, s));
    SPH_HIP_TRY(hipMemcpyAsync(&dmax, w.max_depth, sizeof dmax, hipMemcpyDeviceToHost, s));
    SPH_HIP_TRY(hipStreamSynchronize(s));
    if (nodes_out) *nodes_out = K;
    if (K > cap)
        return fail(SPH_ERR_CAPACITY, "%lld inner nodes exceed capacity %lld", (long long)K,
                    (long long)cap);
    if (dmax > kDepthMax || (K > 0) != (dmax >= 0))
        return fail(SPH_ERR_HIP, "tree bookkeeping: depth %d with %lld nodes", dmax, (long long)K);

    k_items<<<nb, kBlock, 0, s>>>(x, y, z, m, key, idx, w.off, n, w.list, w.it);
    SPH_LAUNCHED();
    for (int d = dmax; d >= 0; --d) {
        k_monopole<<<blocks_for(K), kBlock, 0, s>>>(w.list, K, d, w.it);
        SPH_LAUNCHED();
    }
    const GravConsts k{G, theta * theta, eps, n, n + K};
    const unsigned groups = blocks_for(n, 64);
    if (groups <= kFewGroups)
        k_walk<kWalkWaves><<<groups, 64 * kWalkWaves, 0, s>>>(k, w.box, idx, w.it, w.off, w.cnt, ax,
                                                              ay, az, count);
    else
        k_walk<1><<<groups, 64, 0, s>>>(k, w.box, idx, w.it, w.off, w.cnt, ax, ay, az, count);
    SPH_LAUNCHED();
    return SPH_OK;
}
