// One wavefront of 64 lanes on the CPU, for tests of device code that synchronises inside
// a wavefront only: each lane is a fiber (ucontext) that runs until the next operation
// across lanes, and goes on once all 64 have come to the same one.  Only what the headers
// under test name is here; what they name but the tests never call is declared so that it
// compiles.
#pragma once

#include <ucontext.h>

#include <climits>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#define __host__
#define __device__
#define __global__
#define __shared__ static
#define __launch_bounds__(...)

struct int2 { int x, y; };
struct double2 { double x, y; };
struct float4 { float x, y, z, w; };
struct alignas(32) double4 { double x, y, z, w; };
struct dim3 { unsigned x, y, z; };
inline int2 make_int2(int x, int y) { return {x, y}; }
inline double2 make_double2(double x, double y) { return {x, y}; }
using hipStream_t = void *;
enum hipError_t { hipSuccess };
inline const char *hipGetErrorString(hipError_t) { return ""; }
inline hipError_t hipGetLastError() { return hipSuccess; }

using std::isfinite;
using std::signbit;
template <class T> T min(T a, T b) { return b < a ? b : a; }
template <class T> T max(T a, T b) { return a < b ? b : a; }

namespace wave {

constexpr int kLanes = 64;
struct Wave {
    ucontext_t main, lane[kLanes];
    char *stack = nullptr;
    bool done[kLanes];
    uint64_t value[2][kLanes];  // what each lane brought to this operation and the last one
    int op[kLanes];             // the operation each lane waits at
    int turn[kLanes];           // operations it has passed
    int at = 0;                 // the lane that runs
    unsigned block = 0, wave = 0;
    long turns = 0;
};
inline Wave w;
inline unsigned grid = 0;

// All lanes meet at operation op, each with a value; returns all 64 of them.
inline const uint64_t *meet(int op, uint64_t v) {
    const int me = w.at, p = w.turn[me]++ & 1;
    w.op[me] = op;
    w.value[p][me] = v;
    swapcontext(&w.lane[me], &w.main);
    return w.value[p];
}

// Runs f() as one wavefront; true when every lane returned within `limit` operations,
// false when they had not.  (Lanes at different operations, or some gone while others
// wait, are an error of the code under test.)
template <class F>
bool run(unsigned block, unsigned wave_, long limit, F f) {
    constexpr size_t kStack = 1 << 16;
    if (!w.stack) w.stack = (char *)malloc(kStack * kLanes);
    static F *fn;
    fn = &f;
    w.block = block;
    w.wave = wave_;
    w.turns = 0;
    for (int l = 0; l < kLanes; ++l) {
        w.done[l] = false;
        w.turn[l] = 0;
        getcontext(&w.lane[l]);
        w.lane[l].uc_stack.ss_sp = w.stack + kStack * l;
        w.lane[l].uc_stack.ss_size = kStack;
        w.lane[l].uc_link = &w.main;
        makecontext(&w.lane[l], (void (*)()) + [] {
            const int me = w.at;
            (*fn)();
            w.done[me] = true;
        }, 0);
    }
    for (; w.turns < limit; ++w.turns) {
        for (w.at = 0; w.at < kLanes; ++w.at) swapcontext(&w.main, &w.lane[w.at]);
        int gone = 0;
        for (int l = 0; l < kLanes; ++l) gone += w.done[l];
        if (gone == kLanes) return true;
        for (int l = 0; l < kLanes; ++l)
            if (gone || w.op[l] != w.op[0]) {
                fprintf(stderr, "lanes of a wavefront at different operations\n");
                abort();
            }
    }
    return false;
}

struct ThreadIdx {
    struct { operator unsigned() const { return 64 * w.wave + w.at; } } x;
};
struct BlockIdx {
    struct { operator unsigned() const { return w.block; } } x;
};
struct GridDim {
    struct { operator unsigned() const { return grid; } } x;
};

}  // namespace wave

static wave::ThreadIdx threadIdx;
static wave::BlockIdx blockIdx;
static wave::GridDim gridDim;
static struct { unsigned x; } blockDim{256};

inline unsigned __lane_id() { return (unsigned)wave::w.at; }
inline unsigned long long __ballot(bool p) {
    const uint64_t *v = wave::meet(1, p);
    unsigned long long r = 0;
    for (int l = 0; l < 64; ++l) r |= (unsigned long long)(v[l] != 0) << l;
    return r;
}
template <class T> uint64_t wave_bits(T v) {
    uint64_t b = 0;
    memcpy(&b, &v, sizeof v);
    return b;
}
template <class T> T wave_value(uint64_t b) {
    T v;
    memcpy(&v, &b, sizeof v);
    return v;
}
template <class T> T __shfl(T v, int l) { return wave_value<T>(wave::meet(2, wave_bits(v))[l & 63]); }
template <class T> T __shfl_xor(T v, int o) {
    const int me = wave::w.at;
    return wave_value<T>(wave::meet(3, wave_bits(v))[me ^ o]);
}
template <class T> T __shfl_up(T v, int o) {
    const int me = wave::w.at;
    return wave_value<T>(wave::meet(4, wave_bits(v))[me >= o ? me - o : me]);
}
template <class T> T __shfl_down(T v, int o) {
    const int me = wave::w.at;
    return wave_value<T>(wave::meet(5, wave_bits(v))[me + o < 64 ? me + o : me]);
}
inline int __builtin_amdgcn_readlane(int v, int l) { return (int)wave::meet(6, (uint32_t)v)[l]; }
inline int __builtin_amdgcn_readfirstlane(int v) { return (int)wave::meet(7, (uint32_t)v)[0]; }
inline void __builtin_amdgcn_wave_barrier() { wave::meet(8, 0); }
// row_shr:1..15 and row_bcast:15 and 31, a lane without a source (or in a masked row) keeps old
inline int __builtin_amdgcn_update_dpp(int old, int v, int ctrl, int rows, int, bool) {
    const int me = wave::w.at;
    const uint64_t *a = wave::meet(9, (uint32_t)v);
    if (!(rows >> (me >> 4) & 1)) return old;
    if (ctrl > 0x110 && ctrl < 0x120) return (me & 15) >= ctrl - 0x110 ? (int)a[me - (ctrl - 0x110)] : old;
    if (ctrl == 0x142) return me >= 16 ? (int)a[(me & ~15) - 1] : old;
    if (ctrl == 0x143) return me >= 32 ? (int)a[31] : old;
    abort();
}
inline void __builtin_amdgcn_s_waitcnt(int) {}
inline void __builtin_amdgcn_fence(int, const char *) {}
inline int __popc(uint32_t v) { return __builtin_popcount(v); }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline int __ffsll(long long v) { return __builtin_ffsll(v); }
template <class T> T atomicOr(T *p, T v) {
    const T o = *p;
    *p |= v;
    return o;
}
inline int atomicCAS(int *p, int a, int b) {
    const int o = *p;
    if (o == a) *p = b;
    return o;
}
// declared only
inline void __syncthreads() { abort(); }
int __builtin_amdgcn_ds_bpermute(int, int);
void __builtin_amdgcn_global_load_lds(const void *, void *, int, int, int);
double __builtin_amdgcn_rsq(double);
double __builtin_amdgcn_rcp(double);
float __builtin_amdgcn_rsqf(float);
float __builtin_amdgcn_rcpf(float);
