"""One step of the open faces from the state that the GPU holds, against the
FP64 oracle, to the rounding of what a step stores.

The oracle starts every step from the GPU's own state, so neither the rounding
of an initial state nor that of earlier steps is left to cover.  What remains
of a step:

* FP32 arithmetic: 1e-5 of the node density, as in the other step tests.
* Binary16 storage holds f - w rho(t), each rounded by at most 2^-11 of its
  magnitude; delta is 2^-11 of the largest one in the domain.  The face rules
  read rounded populations and are read by others: a rounding between the
  streaming and the inlet and outlet rules comes out up to 5.4 times as large
  (measured on the oracle over random signs, both lattices, open and partly
  blocked faces; twice that covers aligned signs), the rounded copies of the
  outlet's entering populations, which the oracle holds in full, up to 1.8
  times, and the result is rounded once more: 14 delta.

That is 1.5e-4 in 2-D and 8e-5 in 3-D here; dropping chi, alpha or the inlet
velocity moves populations by 2.6e-3 at the least.
"""
import numpy as np
import pytest

import oracle
from paper_2512_12934_amd import cases

LENGTH = 8


def _open_channel(dim, axis, side, blocked, chi_on=True, alpha_on=True, u_n=0.03):
    """A channel without side walls along ``axis``, its outlet on ``side``;
    the flow slows down towards the outlet, so chi is far from 1."""
    shape = [13, 13 if dim == 2 else 5, 1 if dim == 2 else 6]
    shape[axis] = LENGTH
    periodic = [True, True, True]
    periodic[axis] = False
    c = cases.Case(f"open_axis{axis}_side{side}_blocked{blocked}", dim, tuple(shape), tuple(periodic), (0.1, 0.2), 0.9,
                   solid=np.zeros(int(np.prod(shape)), np.uint8), rho0=None)
    xyz = c.grid()
    flow = xyz[axis] if side == 1 else LENGTH - 1 - xyz[axis]
    across = xyz[1 - axis]
    if blocked:
        c.solid = (((flow == LENGTH - 1) & (across == 3)) | ((flow == LENGTH - 2) & (across == 2))).astype(np.uint8)
    rng = np.random.default_rng(7)
    c.rho0 = np.stack([0.5 + 0.1 * rng.random(c.N), 0.6 + 0.1 * rng.random(c.N)])
    c.u0 = np.zeros((3, c.N))
    c.u0[axis] = (1 if side == 1 else -1) * (0.04 - 0.02 * flow / (LENGTH - 1))
    c.u0[:, c.solid == 1] = 0.0
    hi = tuple(shape)
    c.inlets = [cases.inlet(axis, 1 - side, (0, 0, 0), hi, (0.55, 0.65), u_n, alpha_on)]
    c.outlet = cases.outlet(axis, side, (0, 0, 0), hi, chi_on)
    return c


def _step(c, f, storage):
    """The oracle's step from f: the next state, its diagnostics, the bound on
    a population relative to the node density (per node), and that on u_conv."""
    _, w, _, _ = oracle.tables(c.dim)
    s = oracle.Sim(c)
    s.set_f(f)
    s.step(1)
    fn, d = s.get_f(), s.diag()
    fluid = c.solid == 0
    rho = f.sum(axis=1)
    held = max(np.abs(v - w[None, :, None] * rho[:, None])[:, :, fluid].max() for v in (f, fn))
    face = 14 * held * 2.0 ** -11 if storage == "f16" else 0.0
    return fn, d, 1e-5 + face / fn[:, :, fluid].sum(axis=(0, 1)), 1e-5 + face


def _worst(a, b, tol, fluid):
    """Largest difference of two states as a share of the bound."""
    return (np.abs(a - b)[:, :, fluid].max(axis=(0, 1)) / b[:, :, fluid].sum(axis=(0, 1)) / tol).max()


@pytest.mark.parametrize("dim", [2, 3])
def test_the_bound_catches_a_missing_rule(dim):
    """The oracle without chi, without alpha or with another inlet velocity is
    ten times further from the oracle than the binary16 bound."""
    for axis in range(2):
        for side in (0, 1):
            for blocked in (False, True):
                c = _open_channel(dim, axis, side, blocked)
                f = oracle.Sim(c).get_f()
                fn, d, tol, _ = _step(c, f, "f16")
                assert d["chi"] > 1.4
                for change in ({"chi_on": False}, {"alpha_on": False}, {"u_n": 0.0}):
                    other = _step(_open_channel(dim, axis, side, blocked, **change), f, "f16")[0]
                    assert _worst(other, fn, tol, c.solid == 0) > 10.0, (c.name, change)


@pytest.mark.gpu
@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("chi_on", [True, False])
@pytest.mark.parametrize("dim", [2, 3])
def test_face_steps_to_the_rounding_of_storage(dim, chi_on, storage):
    """State, chi, the flows of eq. (23) and U_c of three steps, each from the
    state the GPU holds, for every orientation of the open faces."""
    from paper_2512_12934_amd.lbm import LBM
    for axis in range(2):
        for side in (0, 1):
            for blocked in (False, True):
                c = _open_channel(dim, axis, side, blocked, chi_on)
                print(f"[gpu] {c.name} {c.n} {storage} chi={chi_on}", flush=True)
                g = LBM(c, storage=storage)
                for t in range(3):
                    fn, d, tol, tol_u = _step(c, g.get_state(), storage)
                    g.step(1)
                    got = g.mass_flux()
                    worst = _worst(g.get_state(), fn, tol, c.solid == 0)
                    print(f"  step {t}: {worst:.2f} of the bound, chi {got['chi']:.6f} / {d['chi']:.6f}, "
                          f"U_c {got['u_conv']:.6f} / {d['u_conv']:.6f}", flush=True)
                    assert worst < 1.0
                    # sums of rho u over the face nodes, each off by FP32 roundings of its density (t = 0 reads
                    # the state as it is; later the outlet column's rounded copies enter Q' through x_{N-1})
                    flow = tol_u * np.abs(c.rho0).sum(axis=0).max() * c.N / LENGTH
                    assert abs(got["q_in"] - d["q_in"]) < flow and abs(got["q_out"] - d["q_out"]) < flow
                    assert abs(got["chi"] - d["chi"]) < 2 * flow / d["q_out"] * max(1.0, d["chi"])
                    assert abs(got["u_conv"] - d["u_conv"]) < tol_u
