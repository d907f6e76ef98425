// The pair list as the pair kernels read it: partner records held in LDS.
//
// The 64 slots of a block lie close together, so their lists name the same partners over
// and over (on a lattice with 57 partners about 460 different slots in 3,500 entries,
// with 250 partners 980 in 14,200).  Over a list with a skin that is not too dense
// (through_window) the FP64 sums therefore load every partner of a block once, into the
// workgroup's LDS, and each lane reads its step's partner from there.  For that
// sph_build_pairs numbers the block's partners ("locals", in the order of the sweep that
// found them; every list is in that order) and leaves, in the part of the block's room that
// its entries do not use,
//   words of a room of b rows of 64
//     [64 b - 128, 64 b)            header: magic, locals, steps; from word 64 on, for
//                                   every round of 32 steps the lowest local named from
//                                   it on and (upper half) one more than the highest
//                                   named up to its end
//     [.. - uni, 64 b - 128)        the locals' slots, uni = 64 floor(b / 8) words
//     below, 128 words a chunk of 4 steps, downwards: the locals of the entries (16 bits
//     each), a lane's four of a chunk in one 8-byte piece
// What is there is a hint: a record is taken from LDS only if the slot it was loaded for
// (tag) is the entry's own slot, else from memory, so that a list without these words,
// or with others, gives the same sums.
#pragma once

#include "common.hpp"
#include "rhs_common.hpp"

namespace sph {

constexpr int kHintMagic = 0x48535057;
constexpr int kHintHeader = 128;       // words
constexpr int kChunkSteps = 4;         // steps whose locals a lane loads at once
constexpr int kRoundSteps = 32;        // steps of a round
constexpr int kMaxRounds = 64;         // rounds a header describes
constexpr int kMaxHintRoom = 1 << 18;  // rows of a room that may hold hints
constexpr int kMaxLocals = 2047;       // locals numbered

struct HintLayout {
    int uni;    // words of the slots of the locals
    int steps;  // most steps that leave the entries clear of the hints (0: no hints)
};

// (slot: the list's entries, whose hints are read 8 bytes at a time)
__host__ __device__ inline HintLayout hint_layout(int64_t room_rows, const int32_t *slot) {
    HintLayout h{0, 0};
    if (room_rows < 8 || room_rows > kMaxHintRoom || ((uintptr_t)slot & 7) != 0) return h;
    h.uni = 64 * (int)(room_rows >> 3);
    const int chunks = (64 * (int)room_rows - kHintHeader - h.uni) / (96 * kChunkSteps);
    h.steps = kChunkSteps * chunks;
    if (h.steps > kRoundSteps * kMaxRounds) h.steps = kRoundSteps * kMaxRounds;
    return h;
}

// Candidates of a slot of a list with this many entries of room, on average: what a slot is
// given room for are the slots of the cells within reach of it, in a set that fills space
// those of the volume that a ball of that reach has swept over by a cell.  (Lattices with 69
// to 278 candidates: 69 to 293.)
inline double mean_candidates(const sph_grid &g, int64_t entries) {
    constexpr double pi = 3.14159265358979323846;
    const double r = g.h + g.skin, a = g.cell, b = r + 0.5 * g.skin;
    const double swept = a * a * a + 6.0 * a * a * b + 3.0 * pi * a * b * b + 4.0 / 3.0 * pi * b * b * b;
    return (double)entries / (double)g.n * (4.0 / 3.0 * pi * r * r * r) / swept;
}

// Whether the FP64 sums over a list with a skin go through the window (k_pairs64_window) or
// are gathered (k_pairs64_list), by how dense the set is (entries: the list's capacity; one
// larger than the list needs costs speed only).  A block of 64 slots with more than about 140
// candidates each names more partners than a window holds.  Up to kManyGroups blocks
// (four a CU) such a block is gathered with the window's LDS unused, which leaves two
// workgroups a CU instead of four; beyond, its window is filled again and again, hidden
// behind the other blocks until the sets are denser still.  The extended terms' window holds
// fewer records, and their kernel has no registers left to read ahead.  us, window and list,
// with a skin of 0.15 spacings:
//                              40,000 particles   80,000       200,000
//   plain     111 candidates   50.0  50.7         68.6  80.4   152.6 168.0
//             142              68.4  60.5         91.2 101.7   194.6 208.1
//             172              82.9  69.7        109.2 118.3   239.0 245.5
//             188, non-uniform 93.8 108.3        170.9 145.6   328.3 324.8  (middle: 90,000)
//             285             121.4 100.6        182.3 177.2   390.4 370.5
//   corrected 142              67.6  60.7         95.0  93.5   203.5 215.9
//             172              84.7  70.0        114.2 108.7   249.6 254.7
//   extended   98              56.0  56.7         86.5  83.8   179.3 185.1
//             113              65.6  64.4        102.5  95.3   222.3 213.2
//   both       77              54.5  55.0         83.4  81.6   174.3 179.3
//              98              58.6  56.9         91.6  84.3   193.4 187.1
// Where no form goes through the window no hints are built: 262,144 non-uniform particles'
// list took 1,014 us with them.
constexpr unsigned kManyGroups = 1024;

inline bool through_window(const sph_grid &g, int64_t entries, bool corr, bool ext) {
    const bool few = (g.n + 63) / 64 <= kManyGroups;
    const double most = ext ? (corr ? 90.0 : 110.0) : few ? 125.0 : corr ? 150.0 : 180.0;
    return g.skin > 0.0 && mean_candidates(g, entries) < most;
}

// A block of the pair list as one wavefront sees it.
struct ListBlock {
    const int32_t *row;  // this lane's entry of step j at row[64 j]
    const int32_t *uni;  // slots of the locals; the lane's chunk c of locals at
                         // reinterpret_cast<const int2 *>(uni) - 64 (c + 1) + lane
    int room, hint_steps, uni_cap;  // steps with room; with room for hints; locals with room
    int cnt, steps;      // this lane's candidates; the block's steps
    int locals;          // 0: no hints
    uint32_t round;      // lane r: round r's lowest local, highest + 1 << 16
};

// A lane's entries of four of its wavefront's steps and their locals.
struct ListChunk {
    int32_t t[kChunkSteps];
    int2 local;
};

// Step i of a wavefront's chunk c: wavefront q of P takes chunks q, q + P, ...
template <int P>
__device__ inline int list_step(int q, int c, int i) {
    return kChunkSteps * (q + P * c) + i;
}

// Its chunk c (steps: those that may be read; what lies past the block's own is unused).
template <int P>
__device__ inline ListChunk list_chunk(const ListBlock &v, int q, int c, int steps) {
    ListChunk r;
    const int lane = __lane_id();  // signed: the hints lie below v.uni
    r.local = make_int2(0, 0);  // (asked for first: it is needed first)
    if (list_step<P>(q, c, 0) < min(steps, v.hint_steps))
        r.local = reinterpret_cast<const int2 *>(v.uni)[lane - 64 * (q + P * c + 1)];
#pragma unroll
    for (int i = 0; i < kChunkSteps; ++i) {
        const int j = list_step<P>(q, c, i);
        r.t[i] = j < steps ? v.row[(int64_t)64 * j] : 0;
    }
    return r;
}

// What a wavefront asks for before it can sweep a block (all of it at once, from the
// block's room alone): the header, the lanes' counts, the slots of its blocks of the first
// window and its first chunk.
template <int P, int W>
struct ListAhead {
    static constexpr int kOwn = (W / 64 + P - 1) / P;  // blocks of the window per wavefront
    ListBlock v;
    int head[3];
    int32_t e[kOwn];
    ListChunk chunk;
};

// (w: the block; s: this lane's slot, act: it exists)
template <int P, int W>
__device__ inline ListAhead<P, W> list_ahead(const GridDev &g, int64_t w, int64_t s, bool act) {
    const int64_t base = g.pl_block[w], end = g.pl_block[w + 1];
    ListAhead<P, W> a;
    ListBlock &v = a.v;
    const int lane = __lane_id();
    const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t room = (end - base) >> 6;
    const HintLayout h = hint_layout(room, g.pl_slot);
    v.row = g.pl_slot + base + lane;
    v.room = (int)min(room, (int64_t)1 << 24);
    v.hint_steps = h.steps;
    v.uni_cap = h.steps > 0 ? h.uni : 0;
    v.round = 0;
    v.uni = g.pl_slot;
    a.head[0] = a.head[1] = a.head[2] = 0;
    v.cnt = act ? g.pl_count[s] : 0;
    if (h.steps > 0) {
        const int32_t *head = g.pl_slot + end - kHintHeader;
        v.uni = head - h.uni;
        v.round = (uint32_t)head[64 + lane];
#pragma unroll
        for (int i = 0; i < 3; ++i) a.head[i] = head[i];
    }
#pragma unroll
    for (int i = 0; i < ListAhead<P, W>::kOwn; ++i) {
        const int u = 64 * (q + i * P) + lane;
        a.e[i] = u < v.uni_cap ? v.uni[u] : -1;
    }
    a.chunk = list_chunk<P>(v, q, 0, v.room);
    return a;
}

// Its steps, and whether its hints hold, once what was asked for has come.
template <int P, int W>
__device__ inline ListBlock list_block(const ListAhead<P, W> &a) {
    ListBlock v = a.v;
    v.steps = list_steps(v.cnt);
    v.locals = a.head[0] == kHintMagic && a.head[2] == v.steps && v.steps <= v.hint_steps &&
                       a.head[1] >= 0 && a.head[1] <= v.uni_cap
                   ? a.head[1]
                   : 0;
    return v;
}

// Place of local l in a window of W records: l mod W for the locals that are numbered, some
// place of the window for any other l >= 0.
template <int W>
__host__ __device__ constexpr int window_place(int l) {
#pragma unroll
    for (int i = 0; i < kMaxLocals / W; ++i) l = l >= W ? l - W : l;
    return l < W ? l : W - 1;
}

// Runs use(j, t, r) for the list steps of wavefront q (list_step): t
// is this lane's entry and r = fetch(at) what stands at the place `at` of the window, where
// the entry's record is if it is resident (tag[at] == t; `at` always lies inside the
// window).  A step is fetched while the one before it is evaluated.  With kMass
// r.m = mass(t) besides, which comes from memory by the entry itself: a chunk's are asked
// for while the chunk before it is evaluated, and its entries a chunk earlier.  The window holds
// W records, in blocks of 64: load(p, e) starts the loads of the 64 records of slots e (one
// per lane) into places 64 p .. 64 p + 63.  Locals go to places local mod W; a block of
// locals is loaded once every step below has been done that may need what it replaces.
// ready() is called once, when the first records have arrived.  Every thread of the workgroup
// calls it; on return the window may still be read by others.
template <int P, int W, bool kMass, class Load, class Mass, class Ready, class Fetch, class Use>
__device__ inline void sweep_window(const ListBlock &v, const ListAhead<P, W> &ahead,
                                    int32_t *tag, int64_t n, Load &&load, Mass &&mass,
                                    Ready &&ready, Fetch &&fetch, Use &&use) {
    static_assert(W % 64 == 0, "the window holds whole blocks of records");
    constexpr int NB = W / 64, kRoundChunks = kRoundSteps / kChunkSteps / P;
    static_assert(kRoundChunks >= 1, "a round is one or more chunks of every wavefront");
    constexpr int kAhead = kMass ? 2 : 1;  // chunks asked for ahead of the one evaluated
    const int lane = __lane_id();
    const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    ListChunk cur = ahead.chunk, next = cur;
    if constexpr (kMass) next = list_chunk<P>(v, q, 1, v.steps);
    const int nblk = (v.locals + 63) >> 6;
    const int rounds = max(1, (v.steps + kRoundSteps - 1) / kRoundSteps);
    auto fill = [&](int k, int e) {  // block k of the locals, e: this lane's slot of it
        if ((uint32_t)e >= (uint64_t)n || 64 * k + lane >= v.locals) e = -1;
        const int p = k % NB;
        tag[64 * p + lane] = e;
        if (k < nblk) load(p, e < 0 ? 0 : e);
    };
    // the first window; places of no local get a tag that matches nothing
#pragma unroll
    for (int i = 0; i < ListAhead<P, W>::kOwn; ++i)
        if (q + i * P < NB) fill(q + i * P, ahead.e[i]);
    double m[kChunkSteps];
    if constexpr (kMass) {
#pragma unroll
        for (int i = 0; i < kChunkSteps; ++i)  // (the first chunk was read up to the room)
            m[i] = mass(list_step<P>(q, 0, i) < v.steps ? cur.t[i] : 0);
    }
    auto place = [&](const ListChunk &c, int i) {
        const int w = i < 2 ? c.local.x : c.local.y;
        return window_place<W>((i & 1) ? (int)((uint32_t)w >> 16) : w & 0xffff);
    };
    int loaded = min(nblk, NB), r0 = 0;
    while (true) {
        wait_vm();
        __syncthreads();
        if (r0 == 0) ready();
        // up to the first round that needs a local not loaded yet
        const unsigned long long open =
            v.locals ? __ballot(lane > r0 && lane < rounds && (int)(v.round >> 16) > 64 * loaded) : 0;
        const int r1 = open ? __ffsll((long long)open) - 1 : rounds;
        int c = kRoundChunks * r0;
        const int c1 = kRoundChunks * r1;
        if (c < c1 && list_step<P>(q, c, 0) < v.steps) {
            auto rec = fetch(place(cur, 0));
            for (; c < c1 && list_step<P>(q, c, 0) < v.steps; ++c) {
                const ListChunk after = list_chunk<P>(v, q, c + kAhead, v.steps);
                double mn[kChunkSteps];
                if constexpr (kMass) {
#pragma unroll
                    for (int i = 0; i < kChunkSteps; ++i) mn[i] = mass(next.t[i]);
                } else {
                    next = after;
                }
#pragma unroll
                for (int i = 0; i < kChunkSteps; ++i) {
                    const auto then = fetch(i + 1 < kChunkSteps ? place(cur, i + 1) : place(next, 0));
                    if constexpr (kMass) rec.m = m[i];
                    use(list_step<P>(q, c, i), cur.t[i], rec);
                    rec = then;
                }
                cur = next;
                if constexpr (kMass) {
                    next = after;
#pragma unroll
                    for (int i = 0; i < kChunkSteps; ++i) m[i] = mn[i];
                }
            }
        }
        if (r1 == rounds) return;
        r0 = r1;
        __syncthreads();  // parts of the window are overwritten next
        const int lo = (__builtin_amdgcn_readlane((int)v.round, r0) & 0xffff) >> 6;
        const int from = max(loaded, lo), top = min(nblk, lo + NB);
        for (int k = from + q; k < top; k += P) fill(k, 64 * k + lane < v.locals ? v.uni[64 * k + lane] : -1);
        loaded = max(loaded, top);
    }
}

// The same steps in the same order for a block without hints: gather(e) starts
// the loads of the 64 records of a step's entries (one per lane) into the wavefront's
// buffer, one step ahead; r = fetch() is this lane's.
template <int P, class Gather, class Fetch, class Use>
__device__ inline void sweep_gather(const ListBlock &v, Gather &&gather, Fetch &&fetch, Use &&use) {
    const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto step = [&](int m) { return list_step<P>(q, m / kChunkSteps, m % kChunkSteps); };
    auto entry = [&](int j) { return j < v.steps ? v.row[(int64_t)64 * j] : 0; };
    int t = entry(step(0)), next = entry(step(1));
    if (step(0) < v.steps) gather(t);
    for (int m = 0; step(m) < v.steps; ++m) {
        wait_vm();
        auto r = fetch();
        wave_sync();  // read before the buffer is filled again
        int tag = t;
        asm volatile("" : "+v"(tag));
        r.tag = tag;
        if (step(m + 1) < v.steps) gather(next);
        const int j = step(m), tj = t;
        t = next;
        next = entry(step(m + 2));
        use(j, tj, r);
    }
}

// The F partial sums per lane of the P wavefronts of a workgroup added in wavefront
// order (bit reproducible), the result in wavefront 0: field f is added by wavefront
// f mod P.  scratch: Cap doubles, taken Cap / (64 P) fields at a time; it may alias a
// window read before the call.  Every thread calls it.
template <int P, int Cap, int F>
__device__ inline void fold_fields(double (&v)[F], double *scratch) {
    constexpr int G = Cap / (64 * P) < F ? Cap / (64 * P) : F;
    static_assert(G >= 1, "scratch too small");
    const int q = threadIdx.x >> 6, lane = __lane_id();
#pragma unroll
    for (int f0 = 0; f0 < F; f0 += G) {
        const int m = f0 + G < F ? G : F - f0;
        __syncthreads();
#pragma unroll
        for (int f = 0; f < m; ++f) scratch[(f * P + q) * 64 + lane] = v[f0 + f];
        __syncthreads();
        for (int f = q; f < m; f += P) {
            double a = scratch[f * P * 64 + lane];
#pragma unroll
            for (int p = 1; p < P; ++p) a += scratch[(f * P + p) * 64 + lane];
            scratch[f * P * 64 + lane] = a;
        }
        __syncthreads();
        if (q == 0) {
#pragma unroll
            for (int f = 0; f < m; ++f) v[f0 + f] = scratch[f * P * 64 + lane];
        }
    }
}

}  // namespace sph
