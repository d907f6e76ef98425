"""A partner's mass enters the sums as it was given, in every FP64 pair kernel.

Clusters of one heavy particle and 24 massless ones, these at 1/2, 1/4, 1/8 and 1/16 of the
support radius h = 1 along the axes: all distances, 1/r and the kernel's values 1/4, 23/32,
235/256 and 2,003/2,048 are exact in 64 bits.  A massless particle's density sum is one
product of the mass and (8 / pi) w, the massless partners adding zeros, and so has one value
in any order and with any contraction.  (The mass formed again from m / rho and rho is
another number for one density in six.)"""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_hints import headers

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1604_03290_amd")

SIGMA = 2.5464790894703255  # 8 / pi
SHAPE = {0.5: 0.25, 0.25: 23 / 32, 0.125: 235 / 256, 0.0625: 2003 / 2048}
PITCH = 2.25  # of the clusters: no partners outside


def clusters(side, seed):
    rng = np.random.default_rng(seed)
    i = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij")).reshape(3, -1) * PITCH
    off, shape = [np.zeros(3)], [1.0]
    for d, w in SHAPE.items():
        for axis in range(3):
            for sign in (-1.0, 1.0):
                off.append(sign * d * np.eye(3)[axis])
                shape.append(w)
    k, nc = len(off), i.shape[1]
    pos = (i[:, :, None] + np.array(off).T[:, None, :]).reshape(3, -1)
    mass = rng.uniform(1.0, 2.0, nc)
    m = np.zeros((nc, k))
    m[:, 0] = mass
    want = mass[:, None] * (SIGMA * np.array(shape))[None, :]
    n = nc * k
    perm = rng.permutation(n)
    take = lambda a: np.ascontiguousarray(a[..., perm])
    return (take(pos), take(rng.normal(size=(3, n))), take(2700.0 * rng.uniform(0.9, 1.1, n)),
            take(1e7 * rng.normal(size=(6, n))), take(m.ravel())), take(want.ravel())


# 3,375 particles: a workgroup of eight wavefronts takes 64 slots; 18,225: of four
@pytest.mark.parametrize("side", [5, 9])
@pytest.mark.parametrize("extra,correction", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("path", ["list", "list with a skin", "cells"])
def test_density_sum_is_the_product(path, extra, correction, side):
    arrays, want = clusters(side, side)
    st = P.ParticleState.from_arrays(*arrays, "cuda")
    skin = 0.05 if path == "list with a skin" else 0.0
    g = P.sph_build_cells(st.pos, 1.0, skin=skin, cells_per_h=1, pairs=path != "cells")
    if path == "list with a skin":
        assert (headers(g) > 0).any()
    params = dict(W.cube(4, 1.0 / 16, 1).params, h=1.0, dmpd=0.4, correction=float(correction))
    if extra:
        params.update(eps_s=0.2, xsph=0.5)
    out = P.sph_rhs(g, st, params, "fp64", extra=extra)
    assert P.workspace_status(out["_ws"]) == 0
    got = out["rho_sum"].cpu().numpy()
    assert np.array_equal(got, want), (np.count_nonzero(got != want), want.size)
