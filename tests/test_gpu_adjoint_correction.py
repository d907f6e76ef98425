"""The corrected adjoint over a pair list against the same straight from the cells.

Both add the same terms, at most a few hundred per slot, in different orders.  As for the
forward sums that is 1e-12 of the largest output; the correction tensor's derivative holds
the inverse of the moment matrix twice, whose condition (up to thirty in a block, at its
edges) multiplies it by up to a thousand: 1e-9."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1604_03290_amd")

DX = 1.0 / 16
CASES = {
    "ragged": (lambda: W.cube(9, DX, 1), 2, 0.0),  # 729: eleven groups and 25 slots
    "groups": (lambda: W.cube(12, DX, 2, shuffle=True), 2, 0.15),  # 1,728: whole groups
    "many": (lambda: W.cube(26, DX, 4), 2, 0.15),  # 275 groups: four wavefronts each, not eight
    "dense": (lambda: W.cube(11, DX, 3, h_over_dx=3.9), 1, 0.3),
}


@pytest.mark.parametrize("xc", [False, True])
@pytest.mark.parametrize("eps_s", [0.0, 0.2])
@pytest.mark.parametrize("eos", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_list_and_cells_agree(name, eos, eps_s, xc):
    make, cells_per_h, skin = CASES[name]
    w = make()
    st = P.ParticleState.from_arrays(w.pos, w.vel, w.rho, w.S, w.m, "cuda")
    p = dict(w.params, correction=1.0, eos=float(eos), eps_s=eps_s, xsph=0.5 if xc else 0.0)
    gen = torch.Generator(device="cuda").manual_seed(5)
    r = lambda *s: torch.randn(*s, dtype=torch.float64, device="cuda", generator=gen)
    cot = dict(acc=r(3, w.n), drho=r(w.n), dS=r(6, w.n), rho_sum=r(w.n))
    if xc:
        cot.update(du=r(w.n), xv=r(3, w.n))
    got = {}
    for pairs in (False, True):
        g = P.sph_build_cells(st.pos, w.h, skin=skin * w.dx, cells_per_h=cells_per_h, pairs=pairs)
        out = P.sph_rhs_adjoint(g, st, p, cot)
        assert P.workspace_status(out["_ws"]) == 0
        got[pairs] = {k: out[k].cpu().numpy() for k in ("pos", "vel", "rho", "S", "mu", "Y0")}
    for k, v in got[False].items():
        assert np.isfinite(v).all(), k
        assert np.abs(got[True][k] - v).max() <= 1e-9 * np.abs(v).max(), k
