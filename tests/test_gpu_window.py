"""The pair kernels' LDS window: the list's hints never change what the entries say.

The list kernels read partner records from LDS where the words sph_build_pairs keeps
behind a group's entries name them, and from memory otherwise.  Each value and each sum is
the same either way, so the outputs have to be bit-identical with those words wiped, filled
with others or absent; and where the entries themselves are changed, the entries count."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1604_03290_amd")

KEYS = ("acc", "drho", "dS", "rho_sum")
# ragged last groups, one group, a set smaller than a group; 57 partners (one window per
# group) and about 250 (several), and a thin sheet (rooms too small for the words); skins in
# particle spacings, 0: a list without the words
CASES = {
    "cube17": (lambda: W.cube(17, 1.0 / 16, 3), 2, 0.15),
    "four": (lambda: W.cube(26, 1.0 / 16, 9), 2, 0.15),  # 275 groups: four wavefronts each, not eight
    "no_skin": (lambda: W.cube(17, 1.0 / 16, 3), 2, 0.0),
    "cube4": (lambda: W.cube(4, 1.0 / 16, 4), 2, 0.15),
    "few": (lambda: W.cube(3, 1.0 / 16, 5).take(np.arange(11)), 1, 0.15),
    "dense": (lambda: W.cube(20, 1.0 / 16, 6, h_over_dx=3.9), 2, 0.01),
    "dense_skin": (lambda: W.cube(14, 1.0 / 16, 7, h_over_dx=3.9, shuffle=True), 1, 0.6),
    "sheet": (lambda: W.cube(30, 1.0 / 16, 8).take(np.arange(900)), 2, 0.15),
}


def built(name):
    make, cells_per_h, skin = CASES[name]
    w = make()
    st = P.ParticleState.from_arrays(w.pos, w.vel, w.rho, w.S, w.m, "cuda")
    return w, st, P.sph_build_cells(st.pos, w.h, skin=skin * w.dx, cells_per_h=cells_per_h, pairs=True)


def rhs(g, st, w, precision, extra):
    p = dict(w.params, eps_s=0.2, xsph=0.5) if extra else w.params
    out = P.sph_rhs(g, st, p, precision, extra=extra)
    assert P.workspace_status(out["_ws"]) == 0
    return {k: out[k].cpu().numpy() for k in KEYS + (("du", "xv") if extra else ())}


def groups(g):
    """Per group: first entry, rows of room, steps."""
    _, count, block_start, slot, _, _ = g.pairs
    b = block_start.cpu().numpy()
    c = np.zeros(64 * (b.size - 1), dtype=np.int64)
    c[:count.numel()] = count.cpu().numpy()
    return b[:-1], np.diff(b) // 64, c.reshape(-1, 64).max(1)


def change(g, how, rng):
    """The words behind the entries wiped, or overwritten (headers kept, or not)."""
    slot = g.pairs[3]
    s = slot.cpu().numpy()
    for first, room, steps in zip(*groups(g)):
        tail = s[first + 64 * steps:first + 64 * room]
        if how == "wiped":
            tail[:] = 0
        elif how == "random":
            tail[:] = rng.integers(-2 ** 31, 2 ** 31, tail.size)
        elif tail.size > 128:  # a header that holds, with other locals and slots
            tail[:-128] = rng.integers(-2 ** 31, 2 ** 31, tail.size - 128)
    slot.copy_(torch.as_tensor(s))


@pytest.mark.parametrize("precision,extra", [("fp64", False), ("fp64", True), ("fp32comp", False)])
@pytest.mark.parametrize("how", ["wiped", "random", "other locals"])
@pytest.mark.parametrize("name", list(CASES))
def test_hints_do_not_change_the_sums(name, how, precision, extra):
    w, st, g = built(name)
    ref = rhs(g, st, w, precision, extra)
    change(g, how, np.random.default_rng(1))
    got = rhs(g, st, w, precision, extra)
    for k in ref:
        assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("name", ["cube17", "dense", "few"])
@pytest.mark.parametrize("offset", [0, 1])
def test_a_list_without_room_behind_its_entries(name, offset):
    """The same entries in rooms of exactly their steps, at any alignment of the array."""
    w, st, g = built(name)
    ref = rhs(g, st, w, "fp64", False)
    out, count, block_start, slot, x0, partners = g.pairs
    first, room, steps = groups(g)
    s = slot.cpu().numpy()
    packed = np.concatenate([s[a:a + 64 * k] for a, k in zip(first, steps)] + [np.zeros(offset, s.dtype)])
    room2 = torch.as_tensor(np.roll(packed, offset).copy()).cuda()
    start2 = torch.as_tensor(np.concatenate([[0], np.cumsum(64 * steps)])).cuda()
    out.slot = room2.data_ptr() + 4 * offset
    out.block_start = start2.data_ptr()
    got = rhs(g, st, w, "fp64", False)
    for k in KEYS:
        assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("fp32comp", 1e-6)])
def test_changed_entries_count(precision, tol):
    """Two of every slot's entries exchanged: the sums in another order (rounding only);
    another list's entries in place: that list's sums."""
    w, st, g = built("cube17")
    ref = rhs(g, st, w, precision, False)
    slot, count = g.pairs[3], g.pairs[1].cpu().numpy()
    s = slot.cpu().numpy()
    for first, _, steps in zip(*groups(g)):
        rows = s[first:first + 64 * steps].reshape(steps, 64)
        lane = np.arange(64)
        last = np.zeros(64, dtype=np.int64)
        block = count[(first_slot := 64 * int(np.searchsorted(groups(g)[0], first))):first_slot + 64]
        last[:block.size] = np.maximum(block - 1, 0)
        rows[0, lane], rows[last, lane] = rows[last, lane].copy(), rows[0, lane].copy()
    slot.copy_(torch.as_tensor(s))
    got = rhs(g, st, w, precision, False)
    for k in KEYS:
        assert np.abs(got[k] - ref[k]).max() <= tol * np.abs(ref[k]).max(), k
