"""The pair sums straight from the cells, against the same sums over a pair list.

Both add the same terms of 64-bit arithmetic, at most a few hundred per slot, in different
orders: 300 terms of 1.1e-16 each, and a sum of magnitudes up to twenty times the largest
output, leave 1e-12 of that output.  The correction tensor inverts a moment matrix, whose
condition (up to a hundred at a surface) multiplies this: 1e-10, on sets that fill space."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1604_03290_amd")

DX = 1.0 / 16


def scattered(n, seed):
    """A cube's particles drawn far apart: each group of slots lies in many tiles."""
    w = W.cube(24, DX, seed)
    return w.take(np.sort(np.random.default_rng(seed).choice(24 ** 3, n, replace=False)))


# one slot, one group less, exactly and more than full; several tiles; more candidates than
# fit the LDS at a time; the last set whose groups have eight wavefronts and the first with
# four; groups swept slot by slot; a single row of cells
CASES = {
    "one": (lambda: W.cube(4, DX, 1).take(np.arange(1)), 2, 0.0),
    "63": (lambda: W.cube(4, DX, 2).take(np.arange(63)), 2, 0.0),
    "64": (lambda: W.cube(4, DX, 3), 1, 0.0),
    "65": (lambda: W.cube(5, DX, 4).take(np.arange(65)), 2, 0.15),
    "tiles": (lambda: W.cube(17, DX, 5, shuffle=True), 2, 0.15),
    "dense": (lambda: W.cube(15, DX, 6, h_over_dx=3.9), 1, 0.5),
    "256 groups": (lambda: W.cube(26, DX, 10).take(np.arange(16384)), 2, 0.0),
    "257 groups": (lambda: W.cube(26, DX, 11).take(np.arange(16385)), 2, 0.15),
    "sheet": (lambda: W.cube(30, DX, 7).take(np.arange(900)), 2, 0.0),
    "scattered": (lambda: scattered(700, 8), 2, 0.0),
    "line": (lambda: W.cube(66, DX, 9).take(np.arange(66)), 2, 0.0),
}


@pytest.mark.parametrize("name,extra,correction",
                         [(c, e, False) for c in CASES for e in (False, True)] +
                         [(c, e, True) for c in ("tiles", "dense", "257 groups") for e in (False, True)])
def test_cells_and_list_agree(name, extra, correction):
    make, cells_per_h, skin = CASES[name]
    w = make()
    st = P.ParticleState.from_arrays(w.pos, w.vel, w.rho, w.S, w.m, "cuda")
    p = dict(w.params, correction=1.0) if correction else dict(w.params)
    if extra:
        p.update(eps_s=0.2, xsph=0.5)
    got = {}
    for pairs in (False, True):
        g = P.sph_build_cells(st.pos, w.h, skin=skin * w.dx, cells_per_h=cells_per_h, pairs=pairs)
        out = P.sph_rhs(g, st, p, "fp64", extra=extra)
        assert P.workspace_status(out["_ws"]) == 0
        got[pairs] = {k: out[k].cpu().numpy() for k in ("acc", "drho", "dS", "rho_sum") + (("du", "xv") if extra else ())}
    for k, v in got[True].items():
        assert np.isfinite(v).all(), k
        assert np.abs(got[False][k] - v).max() <= (1e-10 if correction else 1e-12) * np.abs(v).max(), k
