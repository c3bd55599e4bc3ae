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
# a partner, a block and its neighbours (4 nodes in 3-D; in 2-D 8, of which 6
# are inner ones where the outlet's launch sums eq. 21), thousands
FACES = [("2d", 1), ("2d", 2), ("2d", 5), ("2d", 6), ("2d", 7), ("2d", 8), ("2d", 9), ("2d", 13), ("2d", 2049),
         ("3d", 1), ("3d", 2), ("3d", 3), ("3d", 46)]


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


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("chi_on", [True, False])
@pytest.mark.parametrize("dim", [2, 3])
def test_face_orientations(dim, chi_on, storage):
    """Channels whose faces have no side walls (periodic across, so the first
    and last outlet nodes are neighbours), along either axis and direction, and
    an outlet with solid nodes in it and behind it."""
    n, w = 8, 13
    for axis in range(2):
        for side in (0, 1):
            for blocked in (False, True):
                shape = [w, w if dim == 2 else 5, 1 if dim == 2 else 6]
                shape[axis] = n
                periodic = [True, True, True]
                periodic[axis] = False
                c = cases.Case(f"open_axis{axis}_side{side}_blocked{blocked}", dim, tuple(shape), tuple(periodic),
                               (0.1, 0.2), 0.9, solid=np.zeros(int(np.prod(shape)), np.uint8), rho0=None)
                xyz = c.grid()
                flow = xyz[axis] if side == 1 else n - 1 - xyz[axis]
                across = xyz[1 - axis]
                if blocked:
                    c.solid = (((flow == n - 1) & (across == 3)) | ((flow == n - 2) & (across == 2))).astype(np.uint8)
                rng = np.random.default_rng(7)
                c.rho0 = np.stack([0.5 + 0.1 * rng.random(c.N), 0.6 + 0.1 * rng.random(c.N)])
                c.u0 = np.zeros((3, c.N))
                c.u0[axis] = 0.02 if side == 1 else -0.02
                c.u0[:, c.solid == 1] = 0.0
                hi = tuple(shape)
                c.inlets = [cases.inlet(axis, 1 - side, (0, 0, 0), hi, (0.55, 0.65), 0.02)]
                c.outlet = cases.outlet(axis, side, (0, 0, 0), hi, chi_on)
                assert _step_error(c, storage) < TOL[storage]
                assert _step_error(c, storage, steps=2) < 2 * TOL[storage]


def _components(field, lo):
    """Face-connected components of a boolean [z, y, x] box, by first node of
    the domain whose corner the box's lo is relative to."""
    from scipy import ndimage
    lab, n = ndimage.label(field, structure=ndimage.generate_binary_structure(3, 1))
    out = []
    for j, (sz, sy, sx) in enumerate(ndimage.find_objects(lab), 1):
        zz, yy, xx = np.nonzero(lab[sz, sy, sx] == j)
        zz, yy, xx = zz + sz.start + lo[2], yy + sy.start + lo[1], xx + sx.start + lo[0]
        out.append((xx, yy, zz))
    return out


# rows and boxes around a wave (64 nodes) and a block (256), a box that leaves
# the domain's rim out, more components than are ordered on the device, a
# spiral (a chain as long as the box), one node, nothing
PATTERNS = ["checker", "spiral", "stripes", "comb", "one", "none", "full"]


@pytest.mark.parametrize("layout", ["caller", "face_last"])
@pytest.mark.parametrize("shape", [(3, 3, 1), (63, 5, 1), (65, 66, 1), (257, 37, 1), (130, 129, 1), (5, 3, 4),
                                   (66, 9, 7)])
@pytest.mark.parametrize("pattern", PATTERNS)
def test_label_patterns(pattern, shape, layout):
    """Components and probe counts of planted fields equal a CPU labelling."""
    import torch
    from paper_2512_12934_amd.lbm import LBM
    if layout == "face_last" and shape[2] == 1:
        pytest.skip("a 3-D layout")
    nx, ny, nz = shape
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    if pattern == "checker":
        f = (x + y + z) % 2 == 0
    elif pattern == "spiral":
        f = np.zeros((nz, ny, nx), bool)
        x0, x1, y0, y1 = 0, nx - 1, 0, ny - 1
        while x0 <= x1 and y0 <= y1:
            f[:, y0, max(0, x0 - 1):x1 + 1] = True
            f[:, y0:y1 + 1, x1] = True
            if y1 > y0:
                f[:, y1, x0:x1 + 1] = True
                f[:, min(y0 + 2, y1):y1 + 1, x0] = True
            x0, x1, y0, y1 = x0 + 2, x1 - 2, y0 + 2, y1 - 2
    elif pattern == "stripes":
        f = y % 2 == 0
    elif pattern == "comb":
        f = (x % 2 == 0) | (y == ny - 1)
    elif pattern == "one":
        f = (x == nx // 2) & (y == ny - 1) & (z == 0)
    else:
        f = np.full((nz, ny, nx), pattern == "full")
    dim = 2 if nz == 1 else 3
    rho = np.where(f.reshape(-1), 1.0, 0.2)
    c = cases.Case(f"labels_{pattern}", dim, shape, (True, True, True), (0.1, 0.1), 0.9,
                   solid=np.zeros(f.size, np.uint8), rho0=np.stack([rho, 1.2 - rho]))
    print(f"[gpu] {c.name} {shape} {layout}", flush=True)
    sim = LBM(c, layout=layout)
    boxes = [((0, 0, 0), shape)]
    if min(nx, ny) > 3:
        boxes.append(((1, 1, 0), (nx - 1, ny, nz)))
    for lo, hi in boxes:
        ref = []
        for xx, yy, zz in _components(f[lo[2]:hi[2], lo[1]:hi[1], lo[0]:hi[0]], lo):
            ref.append({"first": int((xx + nx * (yy + ny * zz)).min()), "size": len(xx),
                        "lo": (int(xx.min()), int(yy.min()), int(zz.min())),
                        "hi": (int(xx.max()) + 1, int(yy.max()) + 1, int(zz.max()) + 1)})
        ref.sort(key=lambda r: r["first"])
        got, n = sim.components(0, lo, hi, 0.6, max_out=max(1, len(ref)))
        assert n == len(ref) and got == ref
        if n <= 4096:
            assert sim.components(0, lo, hi, 0.6, max_out=max(1, len(ref)), static=True) == (got, n)
        count = torch.full((1,), -1, dtype=torch.int64, device="cuda:0")
        sim.probe(0, lo, hi, 0.6, count)
        assert int(count) == sum(r["size"] for r in ref)
    # the labelling leaves the state as it was
    before = sim.get_state()
    other = LBM(c, layout=layout)
    assert np.array_equal(before, other.get_state())
    sim.step(2)
    other.step(2)
    assert np.array_equal(sim.get_state(), other.get_state())


# samples around a tile (16), a gradient group (64), the eight groups that run
# at once (512) and a chunk (8192)
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 512, 513, 8192, 8193])
def test_surrogate_gradients(n):
    """Gradient and loss against the FP64 oracle.  An FP32 sum of n terms of
    like size is off by at most n/64 + 64 roundings of 6e-8 of the sum of their
    magnitudes: 1e-4 of the largest gradient covers n = 8193."""
    from oracle import mlp_oracle as mo
    from paper_2512_12934_amd.surrogate import Surrogate
    print(f"[gpu] surrogate gradients n={n}", flush=True)
    rng = np.random.default_rng(n)
    X = rng.uniform(-1, 1, (n, 4)).astype(np.float32)
    Y = np.stack([np.sin(2 * X[:, 0]), np.cos(X[:, 3]) - 0.3 * X[:, 1]], 1).astype(np.float32)
    s = Surrogate(members=2, max_n=n, seed=n)
    g, loss = s.forward_backward(X, Y)
    th = s.get_params().astype(np.float64)
    for m in range(2):
        go = mo.grad(th[m], X, Y, 128)
        assert np.abs(g[m] - go).max() < 1e-4 * np.abs(go).max()
        assert abs(loss[m] - mo.loss(th[m], X, Y, 128)) < 1e-5 * max(1.0, loss[m])
    # a parameter set put in from outside is the one that trains
    s.set_params(s.get_params()[::-1].copy())
    g2, _ = s.forward_backward(X, Y)
    assert np.array_equal(g2, g[::-1])


# members around one pass over them (5), queries around a block (16)
@pytest.mark.parametrize("members", [1, 4, 5, 6, 11, 64])
@pytest.mark.parametrize("n", [1, 16, 17, 250])
def test_surrogate_predict(members, n):
    """Ensemble mean and deviation against the FP64 oracle's BF16 inference
    (2e-3: a layer-1 activation whose FP32 value rounds to the other BF16
    neighbour moves an output by 2^-9 of one weight product)."""
    import torch
    from oracle import mlp_oracle as mo
    from paper_2512_12934_amd.surrogate import Surrogate
    print(f"[gpu] surrogate predict members={members} n={n}", flush=True)
    s = Surrogate(members=members, max_n=16, seed=5)
    X = np.random.default_rng(n).uniform(-1, 1, (n, 4)).astype(np.float32)
    mean, sd, fb = (v.cpu().numpy() for v in s.predict(X, threshold=0.05, out_scale=(0.5, 2.0), out_shift=(1.0, 3.0)))
    mu, so, fo = mo.ensemble(list(s.get_params().astype(np.float64)), X, 128, 0.05, out_scale=(0.5, 2.0),
                             out_shift=(1.0, 3.0))
    assert np.abs(mean - mu).max() < 2e-3 and np.abs(sd - so).max() < 2e-3
    margin = np.abs(so - 0.05 * np.abs(mu)).min(axis=1) > 5e-3
    assert (fb.astype(bool)[margin] == fo[margin]).all()


# boxes below, at and just over the tiles (32 and 64 wide, 8 rows) and the
# sweep windows of the configurations whose ring is filled at once (2-D 8, 10
# and 11, 3-D 7 to 10) and window by window (2-D 0 and 4, 3-D 6); 9 x 9 tiles
# of the work list in blocks
RINGS = [((3, 3, 1), False), ((5, 9, 1), False), ((31, 8, 1), True), ((33, 9, 1), False), ((64, 17, 1), True),
         ((66, 16, 1), False), ((290, 70, 1), True), ((3, 3, 3), False), ((33, 9, 3), False), ((31, 8, 5), False), ((32, 16, 9), True)]


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape,walls", RINGS)
def test_ring_edges(shape, walls, storage):
    dim = 2 if shape[2] == 1 else 3
    c = cases.random_box(shape, seed=sum(shape), dim=dim, periodic=(not walls,) * 3, walls=walls, u_amp=0.01,
                         Gw=(0.05, -0.05) if walls else (0.0, 0.0))
    for cfg in ((0, 4, 8, 10, 11) if dim == 2 else (6, 7, 8, 9, 10, 11)):
        assert _step_error(c, storage, tile_config=cfg) < TOL[storage]


@pytest.mark.parametrize("storage,nz", [("f32", 70), ("f16", 140)])
@pytest.mark.parametrize("walls", [False, True])
def test_large_domain_order(storage, nz, walls):
    """Populations beyond the last level cache: the node update takes its work
    items last to first, with a work list (walls) and without one; in a batch
    it takes the same ones first to last.  Equal to the bit."""
    from paper_2512_12934_amd.lbm import LBM, Batch
    c = cases.random_box((300, 90, nz), seed=3, dim=3, periodic=(not walls,) * 3, walls=walls, u_amp=0.01)
    print(f"[gpu] {c.n} {storage} walls={walls}", flush=True)
    g, b = LBM(c, storage=storage, tile_config=6), Batch([c], storage=storage, tile_config=6)
    g.step(2)
    b.step(2)
    assert np.array_equal(g.get_state(), b.members[0].get_state())


@pytest.mark.parametrize("storage", ["f32", "f16", "f16fixed"])
@pytest.mark.parametrize("shapes", [((20, 30, 1), (500, 500, 1)), ((8, 9, 10), (64, 64, 62))])
def test_default_tiles(shapes, storage):
    """No tile configuration named: the pick goes by size, for a batch by its
    members' total (here another class than its small member's own), and
    changes no bit of the result."""
    from paper_2512_12934_amd.lbm import LBM, Batch
    dim = 2 if shapes[0][2] == 1 else 3
    cs = [cases.random_box(s, seed=5, dim=dim, periodic=(True,) * 3, walls=False, u_amp=0.01) for s in shapes]
    print(f"[gpu] default tiles {shapes} {storage}", flush=True)
    b = Batch(cs, storage=storage, tile_config=-1)
    b.step(2)
    for c, m in zip(cs, b.members):
        got = []
        for cfg in (-1, 0):
            g = LBM(c, storage=storage, tile_config=cfg)
            g.step(2)
            got.append(g.get_state())
        assert np.array_equal(got[0], got[1])
        assert np.array_equal(got[0], m.get_state())


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape,walls", RINGS)
def test_moments_edges(shape, walls, storage):
    """Every value of the caller's buffers is written (zeros on solids and for
    the missing axis of 2-D), rho and u agree with the oracle: the velocity is
    a sum of some 40 populations of at most the density, each off by TOL."""
    import torch
    from paper_2512_12934_amd.lbm import LBM, LBM_OK
    dim = 2 if shape[2] == 1 else 3
    c = cases.random_box(shape, seed=sum(shape), dim=dim, periodic=(not walls,) * 3, walls=walls, u_amp=0.01,
                         Gw=(0.05, -0.05) if walls else (0.0, 0.0))
    s = oracle.Sim(c)
    s.step(2)
    ro, uo, _ = s.moments()
    fluid = c.solid == 0
    for layout in (["caller"] if dim == 2 else ["caller", "face_last"]):
        print(f"[gpu] moments {shape} walls={walls} {storage} {layout}", flush=True)
        g = LBM(c, storage=storage, layout=layout)
        g.step(2)
        rho = torch.full((2, c.N), float("nan"), dtype=torch.float64, device="cuda:0")
        u = torch.full((3, c.N), float("nan"), dtype=torch.float64, device="cuda:0")
        assert g.moments_device(rho, u) == LBM_OK
        rho, u = rho.cpu().numpy(), u.cpu().numpy()
        assert (rho[:, ~fluid] == 0).all() and (u[:, ~fluid] == 0).all() and (u[dim:] == 0).all()
        scale = ro[:, fluid].sum(axis=0)
        assert (np.abs(rho - ro)[:, fluid] / scale).max() < 2 * TOL[storage]
        assert np.abs(u - uo)[:, fluid].max() < 4 * TOL[storage]
        assert np.array_equal(g.moments()[0], rho) and np.array_equal(g.moments()[1], u)


@pytest.mark.parametrize("storage,nz", [("f32", 70), ("f16", 140)])
@pytest.mark.parametrize("walls", [False, True])
def test_large_domain_reversed(storage, nz, walls):
    """As test_large_domain_order with a two-pass tile: only the two-pass node
    update takes its items last to first, and only beyond the 256 MiB of the
    last level cache.  A batch never does.  Equal to the bit."""
    from paper_2512_12934_amd.lbm import LBM, Batch, tile_config_desc
    c = cases.random_box((300, 90, nz), seed=3, dim=3, periodic=(not walls,) * 3, walls=walls, u_amp=0.01)
    assert 2 * 19 * c.N * (4 if storage == "f32" else 2) > 256 << 20
    for cfg in (8, 11):
        assert tile_config_desc(3, cfg)["psrc"] == 1
        print(f"[gpu] {c.n} {storage} walls={walls} tile {cfg}", flush=True)
        g, b = LBM(c, storage=storage, tile_config=cfg), Batch([c], storage=storage, tile_config=cfg)
        g.step(2)
        b.step(2)
        assert np.array_equal(g.get_state(), b.members[0].get_state())


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape,walls", RINGS)
def test_moments_of_the_held_state(shape, walls, storage):
    """rho and u against the oracle on the state that the GPU holds, so that no
    rounding of storage is left to cover: a density is a sum of Q values
    rounded to 2^-24 (19 * 6e-8 of it), a velocity two such sums of signed
    values and a force whose 92 differences of densities carry weights that
    add up to less than 2: below 1e-5 of u's unit with G = 0.9."""
    from paper_2512_12934_amd.lbm import LBM
    dim = 2 if shape[2] == 1 else 3
    c = cases.random_box(shape, seed=sum(shape), dim=dim, periodic=(not walls,) * 3, walls=walls, u_amp=0.01,
                         Gw=(0.05, -0.05) if walls else (0.0, 0.0))
    fluid = c.solid == 0
    g, s = LBM(c, storage=storage), oracle.Sim(c)
    print(f"[gpu] moments of the held state {shape} walls={walls} {storage}", flush=True)
    for steps in (0, 2):
        g.step(steps)
        s.set_f(g.get_state())
        ro, uo, _ = s.moments()
        rho, u = g.moments()
        assert (np.abs(rho - ro)[:, fluid] / ro[:, fluid].sum(axis=0)).max() < 2e-6
        assert np.abs(u - uo)[:, fluid].max() < 1e-5


# a 2-D class of its own (250 to 450 thousand nodes), and domains whose fluid
# fills 64-wide tiles badly
@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape,walls", [((1000, 300, 1), False), ((5000, 65, 1), True), ((33, 8000, 1), True),
                                         ((33, 40000, 1), True), ((16, 200, 200), False), ((70, 70, 70), True)])
def test_chosen_tile_is_near_the_fastest(shape, walls, storage):
    """The tile that is taken where none is named, and by "auto", costs a step
    at most 8% more than the fastest of the shallow ones (choices by class
    were measured at one shape of each and are up to 6% off at others), and
    gives its bits.  Each time is the least of five runs of 32 steps, the tiles
    in turn."""
    import torch
    from paper_2512_12934_amd.lbm import LBM
    dim = 2 if shape[2] == 1 else 3
    c = cases.random_box(shape, seed=3, dim=dim, periodic=(not walls,) * 3, walls=walls, u_amp=0.01)
    print(f"[gpu] chosen tile {shape} walls={walls} {storage}", flush=True)
    sims = {cfg: LBM(c, storage=storage, tile_config=cfg) for cfg in (-1, "auto", 8, 9, 10, 11)}
    cost = {cfg: float("inf") for cfg in sims}
    for g in sims.values():
        g.set_graph_steps(16)
        g.step(32)
    for _ in range(5):
        for cfg, g in sims.items():
            torch.cuda.synchronize()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.step(32)
            b.record()
            torch.cuda.synchronize()
            cost[cfg] = min(cost[cfg], a.elapsed_time(b) / 32 * 1e3)
    states = {cfg: g.get_state() for cfg, g in sims.items() if cfg in (-1, "auto", 8)}
    print("  us per step", {k: round(v, 1) for k, v in cost.items()}, flush=True)
    fastest = min(cost[k] for k in (8, 9, 10, 11))
    for cfg in (-1, "auto"):
        assert cost[cfg] < 1.08 * fastest, cfg
        assert np.array_equal(states[cfg], states[8])
