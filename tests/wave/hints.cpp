// The hint kernel of the pair list, run on the CPU a wavefront at a time (hip/hip_runtime.h
// beside this file) for the test of its bounds.
#include "hints.hpp"

// Hints for the groups of a list, written as sph_build_pairs has them written.  Returns 0,
// or 1 where a wavefront has not ended after `limit` operations across lanes.
extern "C" int hints_run(int64_t n, const int32_t *count, const int64_t *block_start,
                             int32_t *slot, long limit) {
    const int64_t nb = (n + 63) / 64;
    wave::grid = sph::blocks_for(nb, 4);
    for (unsigned b = 0; b < wave::grid; ++b)
        for (unsigned q = 0; q < 4; ++q)
            if (!wave::run(b, q, limit, [&] { sph::k_pl_hints(n, count, block_start, slot); }))
                return 1;
    return 0;
}

// Most places and pages of a wavefront's table, most locals, words of a header, its magic.
extern "C" const int32_t hints_limits[5] = {sph::kPageTable, sph::kMaxPages, sph::kMaxLocals,
                                            sph::kHintHeader, sph::kHintMagic};

// Place of a local in a window of `width` records (-1: no kernel has such a window).
extern "C" int window_place(int width, int local) {
    switch (width) {
    case 576: return sph::window_place<576>(local);
    case 640: return sph::window_place<640>(local);
    case 704: return sph::window_place<704>(local);
    default: return -1;
    }
}

// The workgroup that takes the place of workgroup i of n: in runs of `run`, 0: as the kernels
// over a list have them, -1: as the adjoint's over the cells.
extern "C" int64_t placed(unsigned n, unsigned i, int run) {
    wave::w.block = i;
    return run > 0 ? sph::xcd_block(n, run) : run == 0 ? sph::xcd_list_block(n) : sph::xcd_cell_block(n);
}
