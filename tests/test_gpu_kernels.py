"""Kernels at the sizes where their work split can go wrong, against the FP64
oracle: edges of blocks and waves, remainders, the smallest and the largest
of each range.

Tolerances.  FP32 states after one step: 1e-5 of the node density (an
absolute error of order Q * 30 * 6e-8 per population at worst, as the moments
reach about 30 rho).  Binary16 storage rounds every population once at the
start and once at the end of the step, each by at most 2^-12 of its stored
magnitude (below 1 of the node density), and the collision amplifies a
population's error by at most 2 per moment row: 2e-3 bounds it.
"""
import numpy as np
import pytest

import oracle
from paper_2512_12934_amd import cases

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "f16": 2e-3}


def _step_error(c, storage, steps=1, **kw):
    """Largest error of a population relative to the node density."""
    from paper_2512_12934_amd.lbm import LBM
    print(f"[gpu] {c.name} n={c.n} storage={storage} {kw}", flush=True)
    g = LBM(c, storage=storage, **kw)
    s = oracle.Sim(c)
    g.step(steps)
    s.step(steps)
    fg, fo = g.get_state(), s.get_f()
    fluid = c.solid == 0
    assert np.isfinite(fg[:, :, fluid]).all()
    return (np.abs(fg[:, :, fluid] - fo[:, :, fluid]) / fo[:, :, fluid].sum(axis=(0, 1))).max()


# face nodes per launch: one node, a wave's two nodes in 2-D with and without
# a partner, a block and its neighbours (4 nodes in 3-D, 8 in 2-D), and faces
# wide enough that a wave takes several nodes, with a remainder
FACES = [("2d", 1), ("2d", 2), ("2d", 7), ("2d", 8), ("2d", 9), ("2d", 2048), ("2d", 2049), ("2d", 2083),
         ("3d", 1), ("3d", 2), ("3d", 3), ("3d", 45), ("3d", 46)]


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("kind,width", FACES)
def test_face_nodes(kind, width, storage):
    """Inlet and outlet faces of `width` (2-D) or width^2 (3-D) nodes."""
    if kind == "2d":
        c = cases.channel(7, width, 0.02, dim=2, droplet=(5, width / 2, max(1.5, width / 5)))
    else:
        c = cases.coflow3d(length=7, width=width, inner=max(1, width // 3))
    assert _step_error(c, storage) < TOL[storage]
    # a second step reads what the face kernels of the first one stored
    assert _step_error(c, storage, steps=2) < 2 * TOL[storage]
