"""Hints of a pair list at their limits: the groups that get none because they name too many
pages or slots (tests/test_hints_host.py has the same limits on the CPU), the groups whose
partners do not fit the LDS window at once, and the lists too dense for the window.  The
hints never change a bit of the sums, so the sums are compared, bit for bit, with those of
the same list without them.

Single particles far apart are added to the small dense sets: a launch of more than 1,024
groups with few candidates on average goes through the window with all its groups."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1604_03290_amd")

MAGIC, HEADER = 0x48535057, 128
PLACES, PAGES, LOCALS = 512, 384, 2047


def dust(in_reach):
    """64 single particles over a layer, one in the middle of each of 64 tiles of 4 x 4 cells,
    in reach of in_reach[i] neighbouring slots of the i-th of the 16 cells below.  Each
    cell of the layer holds one page of 16 slots, so that 64 lanes name 64 pages for every
    cell they reach."""
    rng = np.random.default_rng(7)
    pos = []
    for ty in range(4):
        for tx in range(16):
            for i in range(16):
                cx, cy = 4 * tx + i % 4, 4 * ty + i // 4
                far = np.stack([cx + rng.uniform(0.02, 0.98, 16), cy + rng.uniform(0.02, 0.98, 16),
                                rng.uniform(15.01, 15.08, 16)])
                for k in range(in_reach[i]):  # the cell's corner nearest to the particle above
                    corner = [c + (0.95 - 0.01 * k if c % 4 < 2 else 0.05 + 0.01 * k) for c in (cx, cy)]
                    far[:, k] = [*corner, 15.98]
                pos.append(far)
            pos.append(np.array([[4 * tx + 2.0], [4 * ty + 2.0], [17.1]]))
    return np.ascontiguousarray(np.concatenate(pos, axis=1))


def single(n, z0, pitch):
    """Positions of n particles without partners, from z0 on."""
    i = np.arange(n)
    return np.stack([i % 20, i // 20 % 5, i // 100]) * pitch + np.array([[1.0], [1.0], [z0]])


def state(pos, seed):
    rng = np.random.default_rng(seed)
    n = pos.shape[1]
    arrays = (np.ascontiguousarray(pos), rng.normal(size=(3, n)), 2700.0 * rng.uniform(0.99, 1.01, n),
              1e7 * rng.normal(size=(6, n)), rng.uniform(1.0, 2.0, n))
    return P.ParticleState.from_arrays(*arrays, "cuda")


# cells of 1: h + skin = 2; (in reach per cell, most pages after a chunk of four steps)
DUST = {
    "all fit": [2, 2, 1, 1, 1, 1] + [0] * 10,         # 128, 384
    "too many pages": [1] * 8 + [0] * 8,              # 256, 512: the table just full
    "no free place": [2, 2] + [1] * 8 + [0] * 6,      # 128, 384, 640
}


def dust_grid(name):
    pos = dust(DUST[name])
    dusty = pos.shape[1] // 64 - 1  # the dust's group: its blocks of cells follow the layer's
    st = state(np.concatenate([pos, single(66000, 40.0, 2.2)], axis=1), 8)
    params = dict(W.cube(4, 1.0 / 16, 1).params, h=1.9, dmpd=0.8)
    box = (np.zeros(3), np.array([63.9, 15.9, 1500.0]))
    return P.sph_build_cells(st.pos, 1.9, skin=0.1, cells_per_h=2, box=box, pairs=True), st, params, dusty


FORMS = [(False, False), (True, False), (False, True), (True, True)]


def form(params, extra, correction):
    return dict(params, correction=float(correction), **(dict(eps_s=0.2, xsph=0.5) if extra else {}))


def block(side, h_over_dx, skin, lone, seed=3):
    """A block of side^3 particles and so many single ones: grid with its list, state, params."""
    w = W.cube(side, 1.0, seed, h_over_dx=h_over_dx)
    pos = np.concatenate([w.pos, single(lone, 4.0 * side, 1.1 * (w.h + skin))], axis=1) if lone else w.pos
    st = state(pos, seed)
    return P.sph_build_cells(st.pos, w.h, skin=skin, cells_per_h=2, pairs=True), st, w.params


def lists(g):
    """Per group: counts of its slots, rows of its room; and all words."""
    _, count, block_start, slot, _, _ = g.pairs
    b = block_start.cpu().numpy()
    c = np.zeros(64 * (b.size - 1), dtype=np.int64)
    c[:count.numel()] = count.cpu().numpy()
    return c.reshape(-1, 64), b, slot.cpu().numpy()


def named(g, i):
    """Entries (steps, 64) of group i, -1 where a lane's list is over."""
    c, b, s = lists(g)
    steps = c[i].max()
    rows = s[b[i]:b[i] + 64 * steps].reshape(steps, 64).copy()
    rows[np.arange(steps)[:, None] >= c[i][None, :]] = -1
    return rows


def distinct(a):
    return np.unique(a[a >= 0]).size


def headers(g):
    """Number of locals per group (0: no hints)."""
    c, b, s = lists(g)
    out = np.zeros(len(c), dtype=np.int64)
    for i in range(len(c)):
        if b[i + 1] - b[i] >= max(8 * 64, 64 * c[i].max() + HEADER):
            h = s[b[i + 1] - HEADER:b[i + 1]]
            out[i] = h[1] if h[0] == MAGIC and h[2] == c[i].max() else 0
    return out


def wipe(g):
    c, b, s = lists(g)
    for i in range(len(c)):
        s[b[i] + 64 * c[i].max():b[i + 1]] = 0
    g.pairs[3].copy_(torch.as_tensor(s))


def sums(g, st, params, extra=False):
    """FP64 outputs as arrays."""
    out = P.sph_rhs(g, st, params, "fp64", extra=extra)
    assert P.workspace_status(out["_ws"]) == 0
    keys = ("acc", "drho", "dS", "rho_sum") + (("du", "xv") if extra else ())
    return {k: out[k].cpu().numpy() for k in keys}


def same_without_hints(g, st, params, extra=False):
    ref = sums(g, st, params, extra)
    wipe(g)
    got = sums(g, st, params, extra)
    for k in ref:
        assert np.isfinite(ref[k]).all(), k
        assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("name", list(DUST))
def test_pages(name):
    g, st, params, dusty = dust_grid(name)
    rows = named(g, dusty)
    after = [distinct(rows[:k] >> 4) for k in range(4, rows.shape[0] + 4, 4)]
    want = {"all fit": [128, 384], "too many pages": [256, 512], "no free place": [128, 384, 640]}
    assert after == want[name]
    h = headers(g)
    assert (h[dusty] > 0) == (after[-1] <= PAGES)
    assert h[:dusty].any()  # the layer's groups, where their room leaves some
    same_without_hints(g, st, params)


@pytest.mark.parametrize("extra,correction", FORMS)
def test_many_windows(extra, correction):
    """About a thousand partners a slot: groups of up to four windows (576 records with the
    extended terms, 704 without), and groups that name more than 2,047 slots."""
    g, st, params = block(19, 6.2, 0.05, 90000)
    h, c = headers(g), lists(g)[0]
    dense = np.flatnonzero(c.max(1) > 100)
    slots = np.array([distinct(named(g, i)) for i in dense])
    assert not h[dense][slots > LOCALS].any() and (slots > LOCALS).any()
    kept = h[dense][h[dense] > 0]
    assert set(kept) <= set(slots) and (kept > 1920).any() and (kept < 1408).any()
    same_without_hints(g, st, form(params, extra, correction), extra)


@pytest.mark.parametrize("side,h_over_dx,hints", [(12, 2.4, True), (12, 3.9, False), (41, 3.1, True),
                                                  (41, 3.9, False)])
def test_dense_lists_have_none(side, h_over_dx, hints):
    """About 76 candidates a slot, 285, and between them in a launch that fills the chip."""
    g = block(side, h_over_dx, 0.15, 0)[0]
    assert headers(g).any() == hints


# 343 groups (the gathers' plain sums with eight wavefronts a group, the others with four),
# 1,077 (all with four) and, with 113 candidates, the window at 1,024 groups exactly and one more
@pytest.mark.parametrize("side,h_over_dx,take", [(28, 3.9, None), (41, 3.9, None), (41, 2.8, 65536),
                                                 (41, 2.8, 65537)])
@pytest.mark.parametrize("extra,correction", FORMS)
def test_list_and_cells_agree(side, h_over_dx, take, extra, correction):
    """The same terms in other orders, as in the test of the sums from the cells: 1e-12 of the
    largest output, 1e-10 with the correction's inverse."""
    w = W.cube(side, 1.0 / 16, 5, h_over_dx=h_over_dx)
    if take:
        w = w.take(np.arange(take))
    st = P.ParticleState.from_arrays(w.pos, w.vel, w.rho, w.S, w.m, "cuda")
    got = [sums(P.sph_build_cells(st.pos, w.h, skin=0.15 * w.dx, cells_per_h=2, pairs=pairs), st,
                form(w.params, extra, correction), extra) for pairs in (False, True)]
    for k, v in got[1].items():
        assert np.isfinite(v).all(), k
        assert np.abs(got[0][k] - v).max() <= (1e-10 if correction else 1e-12) * np.abs(v).max(), k


@pytest.mark.parametrize("extra", [False, True])
def test_changed_entries_count(extra):
    """Entries of other slots written over the list's, its hints left as they were: the sums
    are those of the entries, as the same list without hints gives them."""
    w = W.cube(17, 1.0 / 16, 3)
    st = P.ParticleState.from_arrays(w.pos, w.vel, w.rho, w.S, w.m, "cuda")
    g = P.sph_build_cells(st.pos, w.h, skin=0.15 * w.dx, cells_per_h=2, pairs=True)
    params = form(w.params, extra, False)
    before, h = sums(g, st, params, extra), headers(g)
    assert (h > 0).all()
    c, b, s = lists(g)
    for i in range(len(c)):  # a slot's second entry over its first
        for lane in np.flatnonzero(c[i] > 1):
            s[b[i] + lane] = s[b[i] + 64 + lane]
    g.pairs[3].copy_(torch.as_tensor(s))
    assert np.array_equal(headers(g), h)
    assert not np.array_equal(sums(g, st, params, extra)["rho_sum"], before["rho_sum"])
    same_without_hints(g, st, params, extra)
