"""Hints of a pair list at their limits: the groups that get none because they name too many
pages or slots (tests/test_hints_host.py has the same limits on the CPU), and the groups whose
partners do not fit the LDS window at once.  The hints never change a bit of the sums, so
every case is compared, bit for bit, with the same list without them."""
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


# cells of 1: h + skin = 2; (in reach per cell, most pages after a chunk of four steps)
DUST = {
    "all fit": [2, 2, 1, 1, 1, 1] + [0] * 10,         # 128, 384
    "too many pages": [1] * 8 + [0] * 8,              # 256, 512: the table just full
    "no free place": [2, 2] + [1] * 8 + [0] * 6,      # 128, 384, 640
}


def dust_grid(name):
    pos = dust(DUST[name])
    n = pos.shape[1]
    rng = np.random.default_rng(8)
    w = W.cube(4, 1.0 / 16, 1)
    params = dict(w.params, h=1.9, dmpd=0.8)
    arrays = (pos, rng.normal(size=(3, n)), 2700.0 * rng.uniform(0.99, 1.01, n),
              1e7 * rng.normal(size=(6, n)), rng.uniform(1.0, 2.0, n))
    st = P.ParticleState.from_arrays(*arrays, "cuda")
    box = (np.zeros(3), np.array([63.9, 15.9, 31.9]))
    g = P.sph_build_cells(st.pos, 1.9, skin=0.1, cells_per_h=2, box=box, pairs=True)
    return g, st, params


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
    g, st, params = dust_grid(name)
    last = g.n // 64 - 1  # the dust, whose blocks of cells lie above the layer's
    rows = named(g, last)
    after = [distinct(rows[:k] >> 4) for k in range(4, rows.shape[0] + 4, 4)]
    want = {"all fit": [128, 384], "too many pages": [256, 512], "no free place": [128, 384, 640]}
    assert after == want[name]
    h = headers(g)
    assert (h[last] > 0) == (after[-1] <= PAGES)
    assert h[:last].any()  # the layer's groups, where their room leaves some
    same_without_hints(g, st, params)


@pytest.mark.parametrize("extra", [False, True])
def test_more_slots_than_numbered(extra):
    """About a thousand partners a slot: some groups name more than 2,047 slots, some fewer."""
    w = W.cube(19, 1.0 / 16, 3, h_over_dx=6.2)
    st = P.ParticleState.from_arrays(w.pos, w.vel, w.rho, w.S, w.m, "cuda")
    g = P.sph_build_cells(st.pos, w.h, skin=0.05 * w.dx, cells_per_h=2, pairs=True)
    h, c = headers(g), lists(g)[0]
    slots = np.array([distinct(named(g, i)) for i in range(len(c))])
    many = slots > LOCALS
    assert many.any() and not many.all()
    assert not h[many].any()
    assert ((h == slots) | (h == 0)).all() and (h > 1500).any()
    same_without_hints(g, st, dict(w.params, eps_s=0.2, xsph=0.5) if extra else w.params, extra)
