// Right-hand side of the SPH solid-body equations.
//
//   prepass   per slot, FP64: gather the particle's state into slot order,
//             pressure (section 2.5.1), von Mises factor (section 2.6),
//             T = sigma / rho^2 with sigma = -p I + f_Y S (section 2.2),
//             V = m / rho; stale-grid and domain checks
//   pairs     per target slot: partner test d^2 < h^2 (section 3.5.2) over the
//             cell rows within reach; density sum (eq. density_by_kernel_sum),
//             velocity gradient L (section 3.1.6), acceleration with the
//             artificial viscosity Pi* (eqs. accel, accel_artvisc, section 3.1.3)
//   postpass  fused into the pair kernel's epilogue, FP64: drho = -rho tr L
//             (eq. continuity_equation_sph), Hooke + Jaumann stress rate
//             (section 2.4), scatter to user order
//
// Cubic B-spline (section 3.1.1) with q = r/h:  W = s/h^3 w(q) and
// W'(r)/r = 6 s/h^5 f(q) with w = 1 - 6q^2 + 6q^3, f = 3q - 2 for q < 1/2 and
// w = 2 (1-q)^3, f = -(1-q)^2 / q for 1/2 <= q < 1, so grad_a W_ab =
// (W'/r)(x_a - x_b) stays finite as r -> 0.
#include <mutex>
#include <type_traits>

#include "common.hpp"
#include "rhs_common.hpp"
#include "timing.hpp"
#include "sweep.hpp"
#include "window.hpp"

namespace sph {
namespace {

// --------------------------------------------------------------- prepass --
// the slot of every user index: inv[perm[s]] = s; mass (null unless asked for): the masses
// m in slot order
__global__ __launch_bounds__(kBlock) void k_invert(const int32_t *__restrict__ perm, int64_t n,
                                                   int32_t *__restrict__ inv,
                                                   const double *__restrict__ m,
                                                   double *__restrict__ mass) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const int32_t a = perm[s];
    inv[a] = (int32_t)s;
    if (mass) mass[s] = m[a];
}

// dd3 / nact (null unless requested): the damage model's rates (section 3.2).  With
// inv (user-order state, its inverse permutation) thread i takes user particle i, so
// the state arrays are read in order and each thread writes its slot's whole 128-byte
// record; without it (slot-ordered state) thread i takes slot i.
__global__ __launch_bounds__(kBlock) void k_prepass(GridDev g, StateDev st, int64_t n, Consts k,
                                                    double *__restrict__ rec,
                                                    int32_t *__restrict__ status, double *dd3,
                                                    int32_t *nact, const int32_t *__restrict__ inv) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t s = inv ? (int64_t)inv[i] : i;
    const int a = inv ? (int)i : io_index(g, s);
    const double S[6] = {st.sxx[a], st.syy[a], st.szz[a], st.sxy[a], st.sxz[a], st.syz[a]};
    const double d = st.d ? st.d[a] : 0.0, rho = st.rho[a], m = st.m[a];
    const double p = write_rec(g, k, s, st.x[a], st.y[a], st.z[a], st.vx[a], st.vy[a], st.vz[a],
                               rho, S, m, rec, status, st.u ? st.u[a] : 0.0, d);
    if (dd3) {
        const double f = (1.0 - d) * yield_factor(k, S);
        const double ph = p >= 0.0 ? p : (1.0 - d) * p;
        const double sig[6] = {f * S[0] - ph, f * S[1] - ph, f * S[2] - ph,
                               f * S[3],      f * S[4],      f * S[5]};
        damage_rate(k, st, n, a, sig, rho, m, d, dd3, nact, status);
    }
}

// FP32 copies of the pair operands (positions stay FP64 for the exact test), 80 bytes:
//   x y | z (vx vy) | (vz rho m V) | (T0 T1 T2 T3) | (T4 T5 c -)
// c being the record's signed sound speed.
__global__ __launch_bounds__(kBlock) void k_narrow(const double *__restrict__ rec, int64_t n,
                                                   float *__restrict__ r32) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const double *r = rec + s * kRec;
    char *o = reinterpret_cast<char *>(r32) + s * kRec32Bytes;
    *reinterpret_cast<double2 *>(o) = make_double2(r[0], r[1]);
    *reinterpret_cast<double *>(o + 16) = r[2];
    *reinterpret_cast<float2 *>(o + 24) = make_float2((float)r[3], (float)r[4]);
    *reinterpret_cast<float4 *>(o + 32) = make_float4((float)r[5], (float)r[6], (float)r[14], (float)r[7]);
    *reinterpret_cast<float4 *>(o + 48) = make_float4((float)r[8], (float)r[9], (float)r[10], (float)r[11]);
    *reinterpret_cast<float4 *>(o + 64) = make_float4((float)r[12], (float)r[13], (float)r[15], 0.0f);
}

// ---------------------------------------------------------- pairs, FP64 --
// The sums of the P wavefronts of a list kernel's workgroup added into wavefront 0
// (fold_fields); the correction's and the extra terms' sums only where they are formed.
template <int P, int Cap, bool kCorr, bool kExt>
__device__ inline void fold_acc64(Acc64 &a, double *scratch) {
    constexpr int F = 13 + (kCorr ? 6 : 0) + (kExt ? 4 : 0);
    double v[F];
    int i = 0;
    v[i++] = a.rs;
#pragma unroll
    for (int c = 0; c < 9; ++c) v[i++] = a.L[c];
    v[i++] = a.ax;
    v[i++] = a.ay;
    v[i++] = a.az;
    if constexpr (kCorr) {
#pragma unroll
        for (int c = 0; c < 6; ++c) v[i++] = a.M[c];
    }
    if constexpr (kExt) {
        v[i++] = a.du;
#pragma unroll
        for (int c = 0; c < 3; ++c) v[i++] = a.xs[c];
    }
    fold_fields<P, Cap>(v, scratch);
    i = 0;
    a.rs = v[i++];
#pragma unroll
    for (int c = 0; c < 9; ++c) a.L[c] = v[i++];
    a.ax = v[i++];
    a.ay = v[i++];
    a.az = v[i++];
    if constexpr (kCorr) {
#pragma unroll
        for (int c = 0; c < 6; ++c) a.M[c] = v[i++];
    }
    if constexpr (kExt) {
        a.du = v[i++];
#pragma unroll
        for (int c = 0; c < 3; ++c) a.xs[c] = v[i++];
    }
}

// FP64 pair sums over the frozen pair list: a workgroup of kSplit wavefronts takes one
// block of 64 slots, wavefront q walking the 64 lists in lock step over steps q,
// q + kSplit, ... and gathering the 64 partner records of each step cooperatively;
// the partial sums are folded into wavefront 0, which runs the postpass.
template <bool kCorr, bool kExt, int P = kSplit>
__global__ __launch_bounds__(64 * P) void k_pairs64_list(GridDev g, int64_t n, Consts k,
                                                              const double *__restrict__ rec,
                                                              StateDev st, OutDev out,
                                                              double *__restrict__ Lout) {
    __shared__ double2 lbuf[P][64 * 8];
    const int q = threadIdx.x >> 6;
    double2 *buf = lbuf[q];
    const int64_t w = xcd_list_block(gridDim.x);
    const int64_t w0 = w * 64;
    if (w0 >= n) return;  // whole workgroup past the end
    const int64_t s = w0 + __lane_id();
    const bool act = s < n;
    const int64_t base = g.pl_block[w];
    const int cnt = act ? g.pl_count[s] : 0;
    const int steps = list_steps(cnt);
    double2 p0 = make_double2(0, 0), p1 = p0, p2 = p0, p3 = p0, p4 = p0, p5 = p0, p6 = p0, p7 = p0;
    if (act) {
        const double2 *ra = rec2(rec, s);
        p0 = ra[0]; p1 = ra[1]; p2 = ra[2]; p3 = ra[3]; p4 = ra[4]; p5 = ra[5]; p6 = ra[6]; p7 = ra[7];
    }
    const double xa = p0.x, ya = p0.y, za = p1.x, vxa = p1.y, vya = p2.x, vza = p2.y;
    const double rho_a = p3.x;
    Acc64 acc;
    if (q == 0) acc.rs = p7.x * k.Wn;  // own term m_a W(0), once
    const double c_a = p7.y;
    const double Ta[6] = {p4.x, p4.y, p5.x, p5.y, p6.x, p6.y};
    const bool tens_a = kExt && signbit(c_a);
    const char *recs = reinterpret_cast<const char *>(rec);
    const int32_t *row = g.pl_slot + base + __lane_id();
    // One step ahead: each lane reads its step-j record into registers, the wavefront
    // syncs, the gathers of step j + P are issued, and step j is evaluated while
    // they are in flight.
    if (q < steps) gather_dma8(recs, kRec * 8, row[(int64_t)q << 6], buf);
    int nxt = q + P < steps ? row[(int64_t)(q + P) << 6] : 0;
    for (int j = q; j < steps; j += P) {
        wait_vm();
        const double2 b0 = dma8_chunk(buf, 0), b1 = dma8_chunk(buf, 1), b2 = dma8_chunk(buf, 2),
                      b3 = dma8_chunk(buf, 3), b4 = dma8_chunk(buf, 4), b5 = dma8_chunk(buf, 5),
                      b6 = dma8_chunk(buf, 6), b7 = dma8_chunk(buf, 7);
        wave_sync();
        if (j + P < steps) {
            gather_dma8(recs, kRec * 8, nxt, buf);
            if (j + 2 * P < steps) nxt = row[(int64_t)(j + 2 * P) << 6];
        }
        if (j < cnt) {
            const double d2 = dist2_exact(xa, ya, za, b0.x, b0.y, b1.x);
            if (d2 < k.h2) {
                const double Tb[6] = {b4.x, b4.y, b5.x, b5.y, b6.x, b6.y};
                pair64<kCorr, kExt>(k, d2, xa - b0.x, ya - b0.y, za - b1.x, b1.y - vxa, b2.x - vya,
                                    b2.y - vza, rho_a, b3.x, p4.x + b4.x, p4.y + b4.y, p5.x + b5.x,
                                    p5.y + b5.y, p6.x + b6.x, p6.y + b6.y, b7.x, b3.y, acc, Ta, Tb,
                                    tens_a, c_a, b7.y);
            }
        }
    }
    fold_acc64<P, P * 64 * 16, kCorr, kExt>(acc, reinterpret_cast<double *>(lbuf));
    if (q != 0 || !act) return;
    const int a = io_index(g, s);
    postpass(k, a, rho_a, acc.L, acc.ax, acc.ay, acc.az, acc.rs, stress_of(st, a).s, out,
             kCorr ? acc.M : nullptr);
    if (kExt) postpass_ext(k, a, acc, st, out);
    if (Lout) store_vgrad<kCorr>(Lout, s, acc.L, acc.M);
}

// The same for a list with a skin, which is built to serve many evaluations and carries
// hints (window.hpp): a block's partner records stand in the workgroup's LDS window, each
// loaded once instead of once per slot that names it.  The window holds the first seven
// chunks of a record, with the extended terms all eight; wavefront q takes every
// kFwdWaves-th chunk of four steps, whose records are read
// from LDS one step ahead.  The mass alone comes from memory by the entry (mass: [n] in slot
// order), two chunks ahead: the address unit is idle here, and an eighth LDS read a step
// costs more (V rho in the mass's place is one rounding off; right-hand side of 262,144
// particles with V rho 160 us, with the mass from memory 165, from the window 171; with the
// extended terms, whose registers do not allow it, 213 with V rho and 223 from the window).
// The kernel above is bound by its gathers (the texture addresser takes 64 B a clock and CU
// at best: 112 B a pair), this one by the pairs' FP64 arithmetic and LDS reads: the whole
// right-hand side of 262,144 particles with a skin of 0.15 spacings 210 us with the gathers,
// 165 here; with the extended terms 272 and 223; two workgroups a CU are enough, since a step
// waits for no memory.
// Without a skin the hints are not built: they cost 85 us on 262,144 particles, more than
// the 45 us of one evaluation, and such a list holds for one set of positions only.
constexpr int kFwdWaves = 4;

template <bool kCorr, bool kExt, int P = kFwdWaves>
__global__ __launch_bounds__(64 * P, 2) void k_pairs64_window(GridDev g, int64_t n, Consts k,
                                                                   const double *__restrict__ rec,
                                                                   StateDev st, OutDev out,
                                                                   double *__restrict__ Lout,
                                                                   const double *__restrict__ mass) {
    constexpr int W = kExt ? 576 : 704;  // two workgroups per CU
    __shared__ double2 ring[W * (kExt ? 8 : 7)];
    double2 *const last = ring + W * 7;  // with kExt the records' last chunks: mass, sound speed
    __shared__ int32_t tag[W];
    const int64_t w = xcd_list_block(gridDim.x);
    const int64_t w0 = w * 64;
    if (w0 >= n) return;  // whole workgroup past the end
    const int64_t s = w0 + __lane_id();
    const bool act = s < n;
    const auto ahead = list_ahead<P, W>(g, w, s, act);
    const double2 *ra = rec2(rec, act ? s : w0);
    const double2 p0 = ra[0], p1 = ra[1], p2 = ra[2], p3 = ra[3], p4 = ra[4], p5 = ra[5],
                  p6 = ra[6], p7 = ra[7];
    const bool first = threadIdx.x < 64 && act;
    const int a = first ? io_index(g, s) : 0;
    Stress S;  // for the postpass, asked for ahead of the sweep
    const ListBlock v = list_block(ahead);
    const double xa = p0.x, ya = p0.y, za = p1.x, vxa = p1.y, vya = p2.x, vza = p2.y;
    const double rho_a = p3.x;
    Acc64 acc;
    if (threadIdx.x < 64) acc.rs = p7.x * k.Wn;  // own term m_a W(0), once
    const double c_a = p7.y;
    const double Ta[6] = {p4.x, p4.y, p5.x, p5.y, p6.x, p6.y};
    const bool tens_a = kExt && signbit(c_a);
    const char *recs = reinterpret_cast<const char *>(rec);
    struct Partner {
        double2 b[7];
        double c, m;
        int32_t tag;
    };
    auto ready = [&] {
        if (first) S = stress_of(st, a);
    };
    auto use = [&](int j, int t, Partner &r) {
        const bool on = j < v.cnt;
        if (__builtin_expect(__ballot(on && r.tag != t) != 0, 0)) {
            if (on) {
                const double2 *m = rec2(rec, t);
#pragma unroll
                for (int i = 0; i < 7; ++i) r.b[i] = m[i];
                if constexpr (kExt) {
                    r.m = m[7].x;
                    r.c = m[7].y;
                }
            }
            wait_vm();  // here, or every step would wait for its prefetch
        }
        const double2 b0 = r.b[0], b1 = r.b[1], b2 = r.b[2], b3 = r.b[3], b4 = r.b[4], b5 = r.b[5],
                      b6 = r.b[6];
        const double d2 = dist2_exact(xa, ya, za, b0.x, b0.y, b1.x);
        if (on && d2 < k.h2) {
            const double Tb[6] = {b4.x, b4.y, b5.x, b5.y, b6.x, b6.y};
            pair64<kCorr, kExt>(k, d2, xa - b0.x, ya - b0.y, za - b1.x, b1.y - vxa, b2.x - vya,
                                b2.y - vza, rho_a, b3.x, p4.x + b4.x, p4.y + b4.y, p5.x + b5.x,
                                p5.y + b5.y, p6.x + b6.x, p6.y + b6.y, r.m, b3.y, acc, Ta, Tb,
                                tens_a, c_a, r.c);
        }
    };
    // A dense group whose partners do not fit the window at once: while the chip is full
    // its reloads and barriers are hidden (300,000 particles with 143 partners 308 us, 397
    // with such groups gathered here); a smaller launch waits for the few densest groups,
    // and then the gathers are the shorter (12,000 to 30,000 non-uniform particles 81 us
    // against 95).
    if (v.locals && (v.locals <= W || gridDim.x > kManyGroups)) {
        sweep_window<P, W, !kExt>(
            v, ahead, tag, n,
            [&](int p, int e) {
                gather_dma<7>(recs, kRec * 8, e, ring + p * 64 * 7);
                if constexpr (kExt) last[64 * p + __lane_id()] = rec2(rec, e)[7];
            },
            [&](int t) { return mass[t]; }, ready,
            [&](int at) {
                Partner r;
#pragma unroll
                for (int i = 0; i < 7; ++i) r.b[i] = ring[7 * at + i];
                if constexpr (kExt) {
                    const double2 b7 = last[at];
                    r.m = b7.x;
                    r.c = b7.y;
                }
                r.tag = tag[at];
                return r;
            },
            use);
    } else {
        ready();
        static_assert(sizeof ring >= P * 64 * 8 * 16, "a step's records for each wavefront");
        double2 *buf = ring + (threadIdx.x >> 6) * 64 * 8;
        sweep_gather<P>(
            v, [&](int e) { gather_dma8(recs, kRec * 8, e, buf); },
            [&] {
                Partner r;
#pragma unroll
                for (int i = 0; i < 7; ++i) r.b[i] = dma8_chunk(buf, i);
                const double2 b7 = dma8_chunk(buf, 7);
                r.m = b7.x;
                r.c = b7.y;
                return r;
            },
            use);
    }
    fold_acc64<P, W * 14, kCorr, kExt>(acc, reinterpret_cast<double *>(ring));
    if (first) {
        postpass(k, a, rho_a, acc.L, acc.ax, acc.ay, acc.az, acc.rs, S.s, out, kCorr ? acc.M : nullptr);
        if (kExt) postpass_ext(k, a, acc, st, out);
        if (Lout) store_vgrad<kCorr>(Lout, s, acc.L, acc.M);
    }
}

// What the pair terms need of a partner's last chunk: its mass and, with the extended
// terms, its signed sound speed.
template <bool kExt>
struct LastChunk {
    double m;
    LastChunk() = default;
    __device__ explicit LastChunk(double2 b) : m(b.x) {}
    __device__ double c() const { return 0.0; }
};
template <>
struct LastChunk<true> {
    double m, s;
    LastChunk() = default;
    __device__ explicit LastChunk(double2 b) : m(b.x), s(b.y) {}
    __device__ double c() const { return s; }
};

// FP64 pair sums straight from the cells: a workgroup of kCellWaves wavefronts takes 64
// slots, in the parts of sweep.hpp.  Their candidates, the slots of the cells around a
// part's box, are culled one per thread against the box widened by h and dealt to the
// wavefronts in turn, each of which has room for kOwn records in LDS; when these are full,
// or the candidates at an end, the records are loaded, each wavefront tests its own for
// all 64 slots (broadcast reads, one bit per candidate and slot) and every slot evaluates
// the partners it was left, whichever they are.  So a step of the evaluation idles only
// the slots that have run out of partners (a lane walking its own slot's cells is idle at
// three candidates of four, some other lane's partners), and a small set still has a
// workgroup per 64 slots.  The tests (12 instructions per candidate and 64 slots) and the
// evaluation each bound it about as much as the search for candidates does.  With one
// slot per lane in workgroups of 256 the whole right-hand side took 241 us for 4,096
// particles, 310 for 110,592 and, with the extended terms, 366; with this 54, 199 and 239.
constexpr int kCellWaves = 4;

template <bool kCorr, bool kExt, int P = kCellWaves>
__global__ __launch_bounds__(64 * P, 2) void k_pairs64_cells(GridDev g, int64_t n, Consts k,
                                                                  const double *__restrict__ rec,
                                                                  StateDev st, OutDev out,
                                                                  double *__restrict__ Lout) {
    using Last = LastChunk<kExt>;
    constexpr int W = kExt ? 576 : 640;  // two workgroups per CU
    constexpr int kOwn = W / P, kWords = (kOwn + 63) / 64;
    constexpr int kBlocks = W / 64, kMine = (kBlocks + P - 1) / P;
    static_assert(64 * P <= W, "a round of candidates fits");
    __shared__ double2 ring[W * 7];
    __shared__ Last last[W];
    __shared__ int32_t tag[W];
    __shared__ int32_t run_s0[kRunCap], run_pre[kRunCap];
    __shared__ int32_t pass[4], kept[2][P];
    __shared__ int32_t self[64];  // places of the group's own slots, -1: not there
    const int lane = __lane_id();
    const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t w0 = xcd_block(gridDim.x) * 64;
    if (w0 >= n) return;  // whole workgroup past the end
    const int64_t s = w0 + lane;
    const bool act = s < n;
    const double2 *ra = rec2(rec, act ? s : w0);  // lanes past n stand on the group's first slot
    const double2 p0 = ra[0], p1 = ra[1], p2 = ra[2], p3 = ra[3], p4 = ra[4], p5 = ra[5],
                  p6 = ra[6], p7 = ra[7];
    const double xa = p0.x, ya = p0.y, za = p1.x, vxa = p1.y, vya = p2.x, vza = p2.y;
    const double rho_a = p3.x;
    Acc64 acc;
    if (q == 0) acc.rs = p7.x * k.Wn;  // own term m_a W(0), once
    const double c_a = p7.y;
    const double Ta[6] = {p4.x, p4.y, p5.x, p5.y, p6.x, p6.y};
    const bool tens_a = kExt && signbit(c_a);
    struct Partner {
        double2 b[7];
        Last l;
    };
    auto use = [&](const Partner &r, bool on) {
        const double2 b0 = r.b[0], b1 = r.b[1], b2 = r.b[2], b3 = r.b[3], b4 = r.b[4], b5 = r.b[5],
                      b6 = r.b[6];
        const double d2 = dist2_exact(xa, ya, za, b0.x, b0.y, b1.x);
        if (on && d2 < k.h2) {
            const double Tb[6] = {b4.x, b4.y, b5.x, b5.y, b6.x, b6.y};
            pair64<kCorr, kExt>(k, d2, xa - b0.x, ya - b0.y, za - b1.x, b1.y - vxa, b2.x - vya,
                                b2.y - vza, rho_a, b3.x, p4.x + b4.x, p4.y + b4.y, p5.x + b5.x,
                                p5.y + b5.y, p6.x + b6.x, p6.y + b6.y, r.l.m, b3.y, acc, Ta, Tb,
                                tens_a, c_a, r.l.c());
        }
    };
    GroupParts parts(g, act, act ? s : w0, xa, ya, za, k.reach);
    while (parts.todo) {
        bool single;
        const bool in = parts.next(g, act, xa, ya, za, k.reach, single);
        const GroupBox &box = parts.box;
        if (single) {  // slot by slot, every P-th candidate a wavefront's
            int i = 0;
            if (in)
                for_each_row(g, xa, ya, za, k.reach, [&](int s0, int s1) {
                    for (int t = s0; t < s1; ++t) {
                        if (t == s || (i++ & (P - 1)) != q) continue;
                        const double2 *rb = rec2(rec, t);
                        Partner r;
                        r.b[0] = rb[0];
                        r.b[1] = rb[1];
                        if (!(dist2_exact(xa, ya, za, r.b[0].x, r.b[0].y, r.b[1].x) < k.h2)) continue;
#pragma unroll
                        for (int c = 2; c < 7; ++c) r.b[c] = rb[c];
                        r.l = Last(rb[7]);
                        use(r, true);
                    }
                });
            continue;
        }
        // the m candidates in tag: candidate i is wavefront i mod P's, at its place i / P
        auto evaluate = [&](int m) {
            if (q == 0) self[lane] = -1;
            __syncthreads();
            int e[kMine];
            bool any[kMine];
#pragma unroll
            for (int i = 0; i < kMine; ++i) {
                const int at = 64 * (q + i * P) + lane;
                const bool there = at < W && P * (at % kOwn) + at / kOwn < m;
                e[i] = there ? tag[at] : (int)w0;
                any[i] = __ballot(there) != 0;
                if (there && (uint32_t)(e[i] - (int)w0) < 64u) self[e[i] - (int)w0] = at;
            }
            Last l[kMine];  // all asked for before any is waited for
#pragma unroll
            for (int i = 0; i < kMine; ++i)
                if (any[i]) {
                    gather_dma<7>(reinterpret_cast<const char *>(rec), kRec * 8, e[i],
                                  ring + (q + i * P) * 64 * 7);
                    l[i] = Last(rec2(rec, e[i])[7]);
                }
#pragma unroll
            for (int i = 0; i < kMine; ++i)
                if (any[i]) last[64 * (q + i * P) + lane] = l[i];
            wait_vm();
            __syncthreads();
            const int mq = m > q ? (m - q + P - 1) / P : 0;
            const double2 *own = ring + q * kOwn * 7;
            uint64_t left[3] = {0, 0, 0};  // this slot's partners among them
            static_assert(kWords <= 3 && kOwn % 4 == 0, "at most three words of bits");
#pragma unroll
            for (int u = 0; u < kWords; ++u) {
                const int bits = min(mq - 64 * u, 64);
                for (int b = 0; b < bits; b += 4) {  // four at a time: their reads overlap
                    double2 b0[4];
                    double z[4];
                    uint32_t hit = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        b0[i] = own[7 * (64 * u + b + i)];
                        z[i] = own[7 * (64 * u + b + i) + 1].x;
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        hit |= (uint32_t)(dist2_exact(xa, ya, za, b0[i].x, b0[i].y, z[i]) < k.h2) << i;
                    left[u] |= (uint64_t)hit << b;
                }
                if (bits < 64) left[u] &= bits > 0 ? (1ull << bits) - 1 : 0;
                const int me = self[lane] - q * kOwn - 64 * u;
                if (me >= 0 && me < 64) left[u] &= ~(1ull << me);
                if (!in) left[u] = 0;
            }
            int first = 0;  // candidate of bit 0 of left[0]
            bool on;
            auto fetch = [&] {  // the next partner (any record where there is none)
                if (left[0] == 0) {
                    left[0] = left[1];
                    left[1] = left[2];
                    left[2] = 0;
                    first += 64;
                }
                if (left[0] == 0) {
                    left[0] = left[1];
                    left[1] = 0;
                    first += 64;
                }
                on = left[0] != 0;
                const int at = on ? first + __builtin_ctzll(left[0]) : 0;
                left[0] &= left[0] - 1;
                Partner r;
#pragma unroll
                for (int c = 0; c < 7; ++c) r.b[c] = own[7 * at + c];
                r.l = last[q * kOwn + at];
                return r;
            };
            Partner r = fetch();
            while (__ballot(on)) {
                if constexpr (kCorr || kExt) {  // (no registers for a record ahead)
                    use(r, on);
                    r = fetch();
                } else {
                    const bool now = on;
                    const Partner then = fetch();
                    use(r, now);
                    r = then;
                }
            }
            __syncthreads();
        };
        const double rb2 = k.h2 * (1.0 + 1e-6);  // far above the rounding of either distance
        int pend = 0, parity = 0;
        const int nrows = box.rows();
        for (int rb = 0, skip = 0; rb < nrows;) {
            if (q == 0) {
                const RunPass p = lay_runs(g, box, parts.tiles == 0, k.reach, rb, skip, run_s0, run_pre);
                if (lane == 0) {
                    pass[0] = rb;
                    pass[1] = skip;
                    pass[2] = p.runs;
                    pass[3] = p.total;
                }
            }
            __syncthreads();
            rb = pass[0];
            skip = pass[1];
            const int runs = pass[2], total = pass[3];
            for (int f0 = 0; f0 < total; f0 += 64 * P) {
                const int f = f0 + threadIdx.x;
                bool keep = false;
                int t = 0;
                if (f < total) {
                    t = slot_of_run(f, runs, run_s0, run_pre);
                    const double2 b0 = rec2(rec, t)[0], b1 = rec2(rec, t)[1];
                    keep = box.dist2(b0.x, b0.y, b1.x) < rb2;
                }
                const unsigned long long mk = __ballot(keep);
                if (lane == 0) kept[parity][q] = __popcll(mk);
                __syncthreads();
                int at = pend, all = 0;
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    if (i < q) at += kept[parity][i];
                    all += kept[parity][i];
                }
                parity ^= 1;  // (written again only after the next barrier)
                at += __popcll(mk & ((1ull << lane) - 1));
                auto put = [&](int i) { tag[i % P * kOwn + i / P] = t; };
                if (keep && at < W) put(at);
                pend += all;
                if (pend >= W) {  // (fewer than W were waiting, at most 64 P <= W came)
                    evaluate(W);
                    if (keep && at >= W) put(at - W);
                    pend -= W;
                }
            }
            __syncthreads();  // the runs are overwritten next
        }
        evaluate(pend);
    }
    fold_acc64<P, W * 14, kCorr, kExt>(acc, reinterpret_cast<double *>(ring));
    if (q != 0 || !act) return;
    const int a = io_index(g, s);
    postpass(k, a, rho_a, acc.L, acc.ax, acc.ay, acc.az, acc.rs, stress_of(st, a).s, out,
             kCorr ? acc.M : nullptr);
    if (kExt) postpass_ext(k, a, acc, st, out);
    if (Lout) store_vgrad<kCorr>(Lout, s, acc.L, acc.M);
}

// ----------------------------------------- pairs, FP32 + Kahan sums --
// unpacked FP32 record of a partner
struct Src32 {
    double x, y, z;
    float vx, vy, vz, rho, m, V, T[6], c;
};

__device__ inline Src32 src32(double2 c0, double2 c1, double2 c2, double2 c3, double2 c4) {
    Src32 r;
    r.x = c0.x;
    r.y = c0.y;
    r.z = c1.x;
    const float2 a = __builtin_bit_cast(float2, c1.y);
    const float4 b = __builtin_bit_cast(float4, c2);
    const float4 t = __builtin_bit_cast(float4, c3);
    const float4 u = __builtin_bit_cast(float4, c4);
    r.vx = a.x; r.vy = a.y; r.vz = b.x; r.rho = b.y; r.m = b.z; r.V = b.w;
    r.T[0] = t.x; r.T[1] = t.y; r.T[2] = t.z; r.T[3] = t.w; r.T[4] = u.x; r.T[5] = u.y;
    r.c = u.z;
    return r;
}

__device__ inline Src32 load32(const float *r32, int64_t s) {
    const double2 *p = reinterpret_cast<const double2 *>(reinterpret_cast<const char *>(r32) +
                                                         s * kRec32Bytes);
    return src32(p[0], p[1], p[2], p[3], p[4]);
}

template <bool kCorr, bool kExt>
__device__ inline void pair32_of(const Consts32 &kf, const Src32 &a, const Src32 &b, double d2,
                                 Acc32 &acc) {
    pair32<kCorr, kExt>(kf, (float)d2, (float)(a.x - b.x), (float)(a.y - b.y),
                        (float)(a.z - b.z), b.vx - a.vx, b.vy - a.vy, b.vz - a.vz, a.rho, b.rho,
                        a.T[0] + b.T[0], a.T[1] + b.T[1], a.T[2] + b.T[2], a.T[3] + b.T[3],
                        a.T[4] + b.T[4], a.T[5] + b.T[5], b.m, b.V, acc, a.T, b.T, a.c, b.c);
}

// the compensated FP32 sums as FP64 values (rs without the particle's own term)
template <bool kCorr, bool kExt>
__device__ inline Acc64 sums_of(const Acc32 &acc) {
    Acc64 v;
    v.rs = acc.rs.value();
#pragma unroll
    for (int c = 0; c < 9; ++c) v.L[c] = acc.L[c].value();
    v.ax = acc.ax.value();
    v.ay = acc.ay.value();
    v.az = acc.az.value();
    if constexpr (kCorr) {
#pragma unroll
        for (int c = 0; c < 6; ++c) v.M[c] = acc.M[c].value();
    }
    if constexpr (kExt) {
        v.du = acc.du.value();
#pragma unroll
        for (int c = 0; c < 3; ++c) v.xs[c] = acc.xs[c].value();
    }
    return v;
}

template <bool kCorr, bool kExt>
__device__ inline void post32(const Consts &k, int a, double rho_a, double m_a, const Acc64 &acc,
                              const Stress &S, const StateDev &st, const OutDev &out, double *Lout,
                              int64_t n, int64_t s) {
    if constexpr (kExt) {
        if (out.du) out.du[a] = 0.5 * acc.du;
        if (out.dx) {
            out.dx[a] = st.vx[a] + k.xsph * acc.xs[0];
            out.dy[a] = st.vy[a] + k.xsph * acc.xs[1];
            out.dz[a] = st.vz[a] + k.xsph * acc.xs[2];
        }
    }
    const double rs = m_a * k.Wn + acc.rs;
    postpass(k, a, rho_a, acc.L, acc.ax, acc.ay, acc.az, rs, S.s, out, kCorr ? acc.M : nullptr);
    if (Lout) store_vgrad<kCorr>(Lout, s, acc.L, acc.M);
}

template <bool kCorr, bool kExt>
__global__ __launch_bounds__(kBlock) void k_pairs32(GridDev g, int64_t n, Consts k,
                                                    const double *__restrict__ rec,
                                                    const float *__restrict__ r32, StateDev st,
                                                    OutDev out, double *__restrict__ Lout) {
    const int64_t s = xcd_block(gridDim.x) * kBlock + threadIdx.x;
    if (s >= n) return;
    const Src32 a = load32(r32, s);
    const double2 p3 = rec2(rec, s)[3], p7 = rec2(rec, s)[7];
    const Consts32 kf = narrow(k);
    Acc32 acc;
    for_each_candidate(g, s, a.x, a.y, a.z, k.reach, [&](int t) {
        const Src32 b = load32(r32, t);
        const double d2 = dist2_exact(a.x, a.y, a.z, b.x, b.y, b.z);
        if (d2 < k.h2) pair32_of<kCorr, kExt>(kf, a, b, d2, acc);
    });
    post32<kCorr, kExt>(k, io_index(g, s), p3.x, p7.x, sums_of<kCorr, kExt>(acc),
                        stress_of(st, io_index(g, s)), st, out, Lout, n, s);
}

// FP32 pair sums over the frozen pair list (cooperative gathers of the 80-byte records)
// the FP32 form over the frozen pair list, kSplit wavefronts per block of 64 slots as
// in the FP64 list kernel (each wavefront's compensated sums folded as FP64 values)
template <bool kCorr, bool kExt>
__global__ __launch_bounds__(64 * kSplit) void k_pairs32_list(GridDev g, int64_t n, Consts k,
                                                              const double *__restrict__ rec,
                                                              const float *__restrict__ r32,
                                                              StateDev st, OutDev out,
                                                              double *__restrict__ Lout) {
    __shared__ double2 lbuf[kSplit][64 * 5];
    const int q = threadIdx.x >> 6;
    double2 *buf = lbuf[q];
    const int64_t w = xcd_list_block(gridDim.x);
    const int64_t w0 = w * 64;
    if (w0 >= n) return;  // whole workgroup past the end
    const int64_t s = w0 + __lane_id();
    const bool act = s < n;
    const int64_t base = g.pl_block[w];
    const int cnt = act ? g.pl_count[s] : 0;
    const int steps = list_steps(cnt);
    const Src32 a = load32(r32, act ? s : w0);
    const Consts32 kf = narrow(k);
    Acc32 acc;
    const char *recs = reinterpret_cast<const char *>(r32);
    const int32_t *row = g.pl_slot + base + __lane_id();
    // one step ahead, as in the FP64 kernel
    if (q < steps) gather_dma<5>(recs, kRec32Bytes, row[(int64_t)q << 6], buf);
    int nxt = q + kSplit < steps ? row[(int64_t)(q + kSplit) << 6] : 0;
    for (int j = q; j < steps; j += kSplit) {
        wait_vm();
        const Src32 b = src32(dma_chunk<5>(buf, 0), dma_chunk<5>(buf, 1), dma_chunk<5>(buf, 2),
                              dma_chunk<5>(buf, 3), dma_chunk<5>(buf, 4));
        wave_sync();
        if (j + kSplit < steps) {
            gather_dma<5>(recs, kRec32Bytes, nxt, buf);
            if (j + 2 * kSplit < steps) nxt = row[(int64_t)(j + 2 * kSplit) << 6];
        }
        if (j < cnt) {
            const double d2 = dist2_exact(a.x, a.y, a.z, b.x, b.y, b.z);
            if (d2 < k.h2) pair32_of<kCorr, kExt>(kf, a, b, d2, acc);
        }
    }
    Acc64 sums = sums_of<kCorr, kExt>(acc);
    fold_acc64<kSplit, kSplit * 64 * 5 * 2, kCorr, kExt>(sums, reinterpret_cast<double *>(lbuf));
    if (q != 0 || !act) return;
    const double2 p3 = rec2(rec, s)[3], p7 = rec2(rec, s)[7];
    const int ia = io_index(g, s);
    post32<kCorr, kExt>(k, ia, p3.x, p7.x, sums, stress_of(st, ia), st, out, Lout, n, s);
}

}  // namespace

int invert_launch(const GridDev &g, int64_t n, int32_t *inv, hipStream_t s) {
    if (!g.io) return SPH_OK;
    k_invert<<<blocks_for(n), kBlock, 0, s>>>(g.io, n, inv, nullptr, nullptr);
    SPH_LAUNCHED();
    return SPH_OK;
}

int prepass_launch(const GridDev &g, const StateDev &st, int64_t n, const Consts &k, double *rec,
                   int32_t *status, hipStream_t s, const OutDev *od, int32_t *inv, double *mass) {
    if (g.io && inv) {
        k_invert<<<blocks_for(n), kBlock, 0, s>>>(g.io, n, inv, st.m, mass);
        SPH_LAUNCHED();
    } else {
        if (mass) return fail(SPH_ERR_NOT_IMPLEMENTED, "masses are put in slot order with inv only");
        inv = nullptr;
    }
    k_prepass<<<blocks_for(n), kBlock, 0, s>>>(g, st, n, k, rec, status, od ? od->dd3 : nullptr,
                                               od ? od->n_act : nullptr, inv);
    SPH_LAUNCHED();
    return SPH_OK;
}

size_t rhs_ws_bytes(int64_t n) {
    Carve c(nullptr);
    c.take<double>((size_t)n * kRec);
    c.take<float>((size_t)n * kRec32);
    c.take<int32_t>(n);
    return c.used;
}

int check_state(const sph_grid *grid, const sph_state *st) {
    if (!st) return fail(SPH_ERR_INVALID_ARG, "state is NULL");
    if (st->n != grid->n) return fail(SPH_ERR_INVALID_ARG, "state n differs from grid n");
    const double *p[] = {st->x,   st->y,   st->z,   st->vx,  st->vy,  st->vz,  st->rho,
                         st->sxx, st->syy, st->szz, st->sxy, st->sxz, st->syz, st->m};
    for (const double *q : p)
        if (!q) return fail(SPH_ERR_INVALID_ARG, "state array is NULL");
    if (!st->flaw_ptr != !st->flaw_eps)
        return fail(SPH_ERR_INVALID_ARG, "flaw_ptr and flaw_eps are given together or not at all");
    return SPH_OK;
}

int check_params(const sph_grid *grid, const sph_params *pr) {
    if (!pr) return fail(SPH_ERR_INVALID_ARG, "params is NULL");
    const double v[] = {pr->h,       pr->rho0,   pr->c,     pr->mu,      pr->Y0,    pr->alpha,
                        pr->beta,    pr->eps_v,  pr->rho_cut, pr->correction, pr->eps_s, pr->n_s,
                        pr->dmpd,    pr->xsph,   pr->eos,   pr->n_M,     pr->a_T,   pr->b_T,
                        pr->A_T,     pr->B_T,    pr->E0_T,  pr->alpha_T, pr->beta_T, pr->E_iv,
                        pr->E_cv};
    for (double q : v)
        if (!std::isfinite(q)) return fail(SPH_ERR_INVALID_ARG, "non-finite parameter");
    if (!(pr->h > 0.0) || !(pr->rho0 > 0.0) || !(pr->c > 0.0))
        return fail(SPH_ERR_INVALID_ARG, "h, rho0 and c must be positive");
    if (pr->mu < 0.0 || !(pr->Y0 > 0.0) || pr->eps_v <= 0.0 || pr->rho_cut < 0.0)
        return fail(SPH_ERR_INVALID_ARG, "mu >= 0, Y0 > 0, eps_v > 0, rho_cut >= 0 required");
    if (pr->h > grid->h) return fail(SPH_ERR_INVALID_ARG, "h exceeds the grid's support radius");
    if (pr->correction != 0.0 && pr->correction != 1.0)
        return fail(SPH_ERR_INVALID_ARG, "correction must be 0 or 1");
    if (pr->eps_s < 0.0 || !(pr->xsph >= 0.0 && pr->xsph <= 1.0))
        return fail(SPH_ERR_INVALID_ARG, "eps_s >= 0 and 0 <= xsph <= 1 required");
    if (pr->eps_s > 0.0 && (!(pr->n_s > 0.0) || !(pr->dmpd > 0.0) || !(pr->dmpd < pr->h)))
        return fail(SPH_ERR_INVALID_ARG, "artificial stress needs n_s > 0 and 0 < dmpd < h");
    if (pr->eos != 0.0 && pr->eos != 1.0 && pr->eos != 2.0)
        return fail(SPH_ERR_INVALID_ARG, "eos must be 0 (liquid), 1 (Murnaghan) or 2 (Tillotson)");
    if (pr->eos == 1.0 && !(pr->n_M > 0.0)) return fail(SPH_ERR_INVALID_ARG, "n_M must be positive");
    if (pr->eos == 2.0 && (!(pr->E0_T > 0.0) || !(pr->E_cv > pr->E_iv) || pr->E_iv < 0.0))
        return fail(SPH_ERR_INVALID_ARG, "Tillotson needs E0_T > 0 and 0 <= E_iv < E_cv");
    return SPH_OK;
}

int check_deriv(const sph_deriv *o) {
    if (!o) return fail(SPH_ERR_INVALID_ARG, "output is NULL");
    const double *p[] = {o->ax, o->ay, o->az, o->drho, o->dsxx, o->dsyy, o->dszz,
                         o->dsxy, o->dsxz, o->dsyz};
    for (const double *q : p)
        if (!q) return fail(SPH_ERR_INVALID_ARG, "output array is NULL");
    if (!(o->dx && o->dy && o->dz) && (o->dx || o->dy || o->dz))
        return fail(SPH_ERR_INVALID_ARG, "dx, dy and dz are given together or not at all");
    if (!o->dd3 != !o->n_act)
        return fail(SPH_ERR_INVALID_ARG, "dd3 and n_act are given together or not at all");
    return SPH_OK;
}

int check_damage(const sph_state *st, const sph_params *pr, const sph_deriv *o) {
    if (o->dd3 && !st->flaw_ptr)
        return fail(SPH_ERR_INVALID_ARG, "damage rates need the flaw lists");
    if (o->dd3 && !(pr->mu > 0.0))
        return fail(SPH_ERR_INVALID_ARG, "damage rates need mu > 0 (Young's modulus)");
    return SPH_OK;
}

// Forward right-hand side on a carved workspace (also used by the leapfrog).
double *rhs_rec_of(Carve c, int64_t n) { return c.take<double>((size_t)n * kRec); }

int rhs_launch(const sph_grid *grid, const sph_state *state, const sph_params *params,
               int precision, const sph_deriv *out, Carve &c, hipStream_t s, double *L_out,
               bool slot_state, bool rec_ready, bool timed) {
    const int64_t n = grid->n;
    GridDev g = grid_dev(grid);
    if (slot_state) g.io = nullptr;
    Consts k = make_consts(*params, g.delta);
    double *rec = rhs_rec_of(c, n);
    c.take<double>((size_t)n * kRec);
    if (out->rec && !rec_ready) rec = out->rec;  // the records go to the caller's buffer
    float *r32 = c.take<float>((size_t)n * kRec32);
    int32_t *inv = c.take<int32_t>(n);
    StateDev st = state_dev(state);
    OutDev od = out_dev(out);
    int rc;
    if (rec_ready && !slot_state)
        return fail(SPH_ERR_NOT_IMPLEMENTED, "records without a prepass need a slot-ordered state");
    if (od.dd3 && rec_ready)
        return fail(SPH_ERR_NOT_IMPLEMENTED, "damage rates need the prepass");
    const bool ext = k.eps_s > 0.0 || od.du || od.dx || k.eos != 0;
    const bool skin = g.pl_count && grid->pairs->skin > 0.0;
    const bool window = skin && through_window(*grid, grid->pairs->capacity, k.corr, ext);
    // masses in slot order for the window kernel, where the FP32 records would be
    const double *mass = state->m;
    double *to = nullptr;
    if (precision == SPH_FP64 && window && !ext && !slot_state)
        mass = to = reinterpret_cast<double *>(r32);
    if (!rec_ready && (rc = prepass_launch(g, st, n, k, rec, c.status(), s, &od, inv, to))) return rc;
    if (precision == SPH_FP64) {
        TimedRegion t(timed ? "pairs_fp64" : nullptr, s);
        auto launch = [&](auto corr, auto extra) {
            constexpr bool C = decltype(corr)::value, E = decltype(extra)::value;
            auto with = [&](auto waves) {
                constexpr int P = decltype(waves)::value;
                const dim3 gb(blocks_for(n, 64)), tb(64 * P);
                if (window)
                    k_pairs64_window<C, E, P><<<gb, tb, 0, s>>>(g, n, k, rec, st, od, L_out, mass);
                else if (g.pl_count)
                    k_pairs64_list<C, E, P><<<gb, tb, 0, s>>>(g, n, k, rec, st, od, L_out);
                else
                    k_pairs64_cells<C, E, P><<<gb, tb, 0, s>>>(g, n, k, rec, st, od, L_out);
            };
            static_assert(kFwdWaves == kSplit && kCellWaves == kSplit, "one choice for all three");
            // A dense list's plain sums keep eight wavefronts up to four blocks a CU: with
            // four all blocks stand on the CUs from the start, and the launch waits for the
            // CU with the most dense ones.  (us with four and eight: 20,000 non-uniform
            // particles 61 and 50, 40,000 108 and 93, 50,000 109 and 113, 65,000 140 and
            // 120; 64,000 with 285 candidates 129 and 130; with the extended terms 40,000
            // with 142 candidates 77 and 84: their eight wavefronts leave one workgroup a CU.)
            const unsigned few = skin && !window && !C && !E ? kManyGroups : kFewBlocks;
            if (blocks_for(n, 64) <= few)
                with(std::integral_constant<int, 2 * kSplit>{});
            else
                with(std::integral_constant<int, kSplit>{});
        };
        using T = std::true_type;
        using F = std::false_type;
        if (k.corr && ext)
            launch(T{}, T{});
        else if (k.corr)
            launch(T{}, F{});
        else if (ext)
            launch(F{}, T{});
        else
            launch(F{}, F{});
        SPH_LAUNCHED();
    } else {
        k_narrow<<<blocks_for(n), kBlock, 0, s>>>(rec, n, r32);
        SPH_LAUNCHED();
        TimedRegion t(timed ? "pairs_fp32comp" : nullptr, s);
        const dim3 gb(blocks_for(n)), tb(kBlock);
        auto launch = [&](auto corr, auto extra) {
            constexpr bool C = decltype(corr)::value, E = decltype(extra)::value;
            if (g.pl_count)
                k_pairs32_list<C, E><<<blocks_for(n, 64), 64 * kSplit, 0, s>>>(g, n, k, rec, r32,
                                                                                 st, od, L_out);
            else
                k_pairs32<C, E><<<gb, tb, 0, s>>>(g, n, k, rec, r32, st, od, L_out);
        };
        using T = std::true_type;
        using F = std::false_type;
        if (k.corr && ext)
            launch(T{}, T{});
        else if (k.corr)
            launch(T{}, F{});
        else if (ext)
            launch(F{}, T{});
        else
            launch(F{}, F{});
        SPH_LAUNCHED();
    }
    return SPH_OK;
}

// ------------------------------------------------ the allocation-free variant --
// Scratch of sph_rhs_noalloc: the workspace of sph_rhs for up to kNoallocMaxN
// particles (status word, FP64 operand records, FP32 records), held by every device
// the library runs on until the process ends.
constexpr int64_t kNoallocMaxN = SPH_NOALLOC_MAX_N;
constexpr size_t kNoallocBytes = kAlign + (size_t)kNoallocMaxN * kRec * sizeof(double) +
                                 (size_t)kNoallocMaxN * kRec32 * sizeof(float) +
                                 (size_t)kNoallocMaxN * sizeof(int32_t);
static_assert(kNoallocMaxN % 64 == 0, "record arrays stay 256-byte aligned");
__device__ __align__(256) unsigned char scratch[kNoallocBytes];

namespace {

// Device address of this device's copy of `scratch` (the array's name is only a
// host-side stand-in in host code), looked up once per device with that device current.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void **out) {
    int dev = -1;
    SPH_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(SPH_ERR_INVALID_ARG, "device %d beyond the %d the library tracks", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        SPH_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(SPH_ERR_HIP, "hipGetSymbolAddress returned no address for the scratch");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return SPH_OK;
}

__global__ void k_copy_status(const int32_t *__restrict__ from, int32_t *__restrict__ to) { *to = *from; }

}  // namespace

}  // namespace sph

using namespace sph;

extern "C" int sph_rhs_noalloc(const sph_grid *grid, const sph_state *state,
                               const sph_params *params, int precision, const sph_deriv *out,
                               int32_t *status, void *stream) {
    clear_error();
    int rc;
    if ((rc = check_grid(grid)) || (rc = check_state(grid, state)) ||
        (rc = check_params(grid, params)) || (rc = check_deriv(out)) ||
        (rc = check_damage(state, params, out)))
        return rc;
    if (precision != SPH_FP64 && precision != SPH_FP32_COMP)
        return fail(SPH_ERR_INVALID_ARG, "unknown precision %d", precision);
    if (out->vgrad && precision != SPH_FP64)
        return fail(SPH_ERR_INVALID_ARG, "vgrad is written by the FP64 form only");
    if (grid->n > kNoallocMaxN)
        return fail(SPH_ERR_CAPACITY, "sph_rhs_noalloc serves at most %lld particles (%lld given)",
                    (long long)kNoallocMaxN, (long long)grid->n);
    if (rhs_ws_bytes(grid->n) > kNoallocBytes)
        return fail(SPH_ERR_CAPACITY, "scratch smaller than the workspace of %lld particles",
                    (long long)grid->n);
    void *ws = nullptr;
    if ((rc = scratch_of_current_device(&ws))) return rc;
    hipStream_t s = (hipStream_t)stream;
    if ((rc = clear_status(ws, s))) return rc;
    Carve c(ws);
    if ((rc = rhs_launch(grid, state, params, precision, out, c, s, out->vgrad, false, false, false)))
        return rc;
    if (status) {
        k_copy_status<<<1, 1, 0, s>>>(reinterpret_cast<const int32_t *>(ws), status);
        SPH_LAUNCHED();
    }
    return SPH_OK;
}

extern "C" int sph_rhs(const sph_grid *grid, const sph_state *state, const sph_params *params,
                       int precision, const sph_deriv *out, void *ws, size_t ws_bytes,
                       void *stream) {
    clear_error();
    int rc;
    if ((rc = check_grid(grid)) || (rc = check_state(grid, state)) ||
        (rc = check_params(grid, params)) || (rc = check_deriv(out)) ||
        (rc = check_damage(state, params, out)))
        return rc;
    if (precision != SPH_FP64 && precision != SPH_FP32_COMP)
        return fail(SPH_ERR_INVALID_ARG, "unknown precision %d", precision);
    if (out->vgrad && precision != SPH_FP64)
        return fail(SPH_ERR_INVALID_ARG, "vgrad is written by the FP64 form only");
    if (!ws) return fail(SPH_ERR_INVALID_ARG, "workspace is NULL");
    const size_t need = rhs_ws_bytes(grid->n);
    if (ws_bytes < need) return fail(SPH_ERR_WORKSPACE, "workspace %zu < %zu bytes", ws_bytes, need);
    hipStream_t s = (hipStream_t)stream;
    if ((rc = clear_status(ws, s))) return rc;
    Carve c(ws);
    return rhs_launch(grid, state, params, precision, out, c, s, out->vgrad);
}
