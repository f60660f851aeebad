"""Kernel variants at the sizes where their dispatch or their tiling can go
wrong, against the FP64 oracle on identical seeded inputs."""
import numpy as np
import pytest

from workloads import fields as F
from workloads import meshes as MM

from oracle import mlp_oracle as M

from test_gpu_implicit import dia_pair
from test_gpu_learned import dev, params, to_bits
from test_gpu_parity import fieldrel, make_pair, random_tree, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def avs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_05645_amd import avs as mod
    return mod


GAS = dict(R=1.0, Pr=2 / 3, omega=0.81, mu_ref=0.02, T_ref=1.0, model=1)


@pytest.mark.parametrize("nx,ny,diatomic", [(5, 1, False), (5, 1, True), (1, 3, False), (4, 3, True)])
def test_repeated_colour_turns(avs, nx, ny, diatomic):
    """Consecutive turns of one colour taken in one launch: cells that read
    their own increment (walls in x, a one-cell periodic axis in y) are
    iterated, the others are not; three sweeps of each kind, to rounding
    (1e-11 as the other implicit tests)."""
    mesh = MM.box2d(nx, ny, periodic=(False, True), sides=dict(left=0, right=0),
                    bcs=[(MM.WALL, (1.0, 0.0, 0.1, 1.1))])
    vs = dict(dim=2, lo=(-6, -6), hi=(6, 6), base=(8, 8), max_level=1)
    prim = F.perturbed_uniform(mesh['ncells'], 2, 11, amp=0.1, uamp=0.3)
    dt = 4.0 * F._cfl_dt(mesh, 1.0, (6.0, 6.0))
    tree = random_tree(vs, 12, 1)
    if diatomic:
        p5 = np.concatenate([prim, 0.9 * prim[:, -1:]], 1)
        cs, dia, o = dia_pair(avs, mesh, vs, GAS, dt, p5, tree)
        dia.step_implicit(2, 3, 3)
        o.step_implicit(2, 3, 3)
        v, W = dia.get_state()
    else:
        cs, o = make_pair(avs, mesh, vs, GAS, dt, prim, tree=tree, noise=0.02, seed=13)
        cs.step_implicit(2, 3, 3)
        o.step_implicit(2, 3, 3)
        v, W = cs.get_state()
    assert rel(v, o.phi) < 1e-11 and rel(W, o.W) < 1e-11


@pytest.mark.parametrize("nx,ny,base,levels,prec", [
    (9, 7, 8, 2, 0),      # 63, 64 and 65 cells
    (8, 8, 8, 2, 0),
    (13, 5, 8, 2, 0),
    (3, 2, 72, 0, 0),     # the largest tables that the lanes would take,
    (3, 2, 73, 0, 0),     # and beyond: a workgroup per cell (few cells)
    (5, 4, 16, 3, 1),     # FP32
    (3, 3, 5, 0, 0),      # fewer leaves than lanes
    (3, 3, 8, 0, 0),      # one leaf per lane
    (3, 3, 38, 0, 0),     # both sides of pass C's 6 KiB of tables, four waves per cell
    (3, 3, 40, 0, 0),
    (3, 3, 38, 0, 1),
    (3, 3, 40, 0, 1),
    (27, 27, 5, 1, 0),    # 1485 faces: a lane per face, 13 in the last group
    (27, 28, 5, 1, 0),    # 1539 faces: three in the last group
    (45, 23, 8, 0, 1),
    (33, 33, 40, 0, 0),   # 2211 faces, tables of 80 entries
])
def test_lane_groups(avs, nx, ny, base, levels, prec):
    """Small and ragged sizes in whatever forms the rules give them (the forms
    themselves are held by test_gpu_forms): a lane or a workgroup per cell and
    per face, one or four waves per cell in pass C; two explicit steps with
    walls (FP64 to 1e-12 per step as the other step tests; FP32 1e-5 of the
    field)."""
    mesh = MM.box2d(nx, ny, periodic=(True, False), sides=dict(bottom=0, top=0),
                    bcs=[(MM.WALL, (1.0, 0.1, 0.0, 1.1))])
    vs = dict(dim=2, lo=(-6, -6), hi=(6, 6), base=(base, base), max_level=levels)
    prim = F.perturbed_uniform(mesh['ncells'], 2, 21, amp=0.1, uamp=0.3)
    cs, o = make_pair(avs, mesh, vs, GAS, F._cfl_dt(mesh, 0.5, (6.0, 6.0)), prim, tree=random_tree(vs, 22, levels),
                      noise=0.02, seed=23, precision=prec)
    cs.step(2)
    o.step(2)
    v, W = cs.get_state()
    if prec:
        assert fieldrel(W, o.W) < 1e-5 and fieldrel(v, o.phi) < 1e-5
    else:
        assert rel(v, o.phi) < 2e-12 and rel(W, o.W) < 2e-12


@pytest.mark.parametrize("prec", [0, 1])
def test_lane_groups_3d(avs, prec):
    mesh = MM.box3d(5, 3, 5)
    vs = dict(dim=3, lo=(-5.0,) * 3, hi=(5.0,) * 3, base=(5, 5, 5), max_level=2)
    prim = F.perturbed_uniform(mesh['ncells'], 3, 31, amp=0.1, uamp=0.3)
    cs, o = make_pair(avs, mesh, vs, GAS, F._cfl_dt(mesh, 0.5, (5.0,) * 3), prim, tree=random_tree(vs, 32, 2),
                      noise=0.02, seed=33, precision=prec)
    cs.step(1)
    o.step(1)
    v, W = cs.get_state()
    tol = 1e-5 if prec else 1e-12
    assert fieldrel(v, o.phi) < tol and fieldrel(W, o.W) < tol


@pytest.mark.parametrize("shape,prec", [((5, 3, 5), 0), ((8, 8, 9), 0), ((8, 8, 9), 1)])
def test_leaf_shares(avs, shape, prec):
    """Few cells and many leaves on small tables, where the rules weigh split
    leaves against a workgroup per cell and per four faces."""
    mesh = MM.box3d(*shape)
    vs = dict(dim=3, lo=(-5.0,) * 3, hi=(5.0,) * 3, base=(18, 18, 18), max_level=0)
    prim = F.perturbed_uniform(mesh['ncells'], 3, 81, amp=0.1, uamp=0.3)
    cs, o = make_pair(avs, mesh, vs, GAS, F._cfl_dt(mesh, 0.5, (5.0,) * 3), prim, noise=0.02, seed=83, precision=prec)
    cs.step(1)
    o.step(1)
    v, W = cs.get_state()
    tol = 1e-5 if prec else 1e-12
    assert fieldrel(v, o.phi) < tol and fieldrel(W, o.W) < tol


@pytest.mark.parametrize("n", [1, 63, 65, 64 * 32, 64 * 33 + 1])
def test_gradient_tile_remainders(avs, n):
    """The network's gradient over batches that end inside a tile of 64 rows
    and whose tiles end inside the reduction's group of 32 (tolerances of the
    larger batch's test: a bfloat16 rounding may fall the other way)."""
    rng = np.random.default_rng(n)
    p = params(41)
    mlp = avs.Mlp(p, max_batch=n)
    X = np.zeros((n, 32))
    X[:, :28] = M.bf16_round(rng.uniform(-1.5, 1.5, (n, 28)))
    flags = rng.integers(-1, 2, n).astype(np.int8)
    g, loss = mlp.grad(dev(to_bits(X)), dev(flags))
    lr, gr = M.loss_and_grad(p, X[:, :28], M.labels_from_flags(flags))
    assert abs(loss - lr) <= 1e-5 * abs(lr)
    G = g.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(G - gr) <= 1e-3 * np.linalg.norm(gr)


@pytest.mark.parametrize("D,base,levels,wall", [
    (2, 8, 4, True),
    (2, 8, 6, True),     # interface tables beyond 64 KiB of LDS
    (2, 3, 1, True),     # fewer leaves than threads
    (2, 90, 0, False),   # one chunk of the moment partials (8100 leaves)
    (2, 91, 0, True),    # two chunks of the moment partials (8281 leaves)
    (3, 4, 2, True),
    (3, 5, 6, False),
])
def test_diatomic_sizes(avs, D, base, levels, wall):
    """Diatomic steps with small and large interface tables, one and two
    chunks of face-moment partials, an odd number of faces, with and without
    walls: two explicit steps and one implicit step (1e-12 per explicit step
    and 1e-11 after the implicit one, as the other diatomic tests)."""
    if D == 2:
        mesh = MM.box2d(5, 3, periodic=(True, not wall), sides=dict(bottom=0, top=0) if wall else None,
                        bcs=[(MM.WALL, (1.0, 0.1, 0.0, 1.1))] if wall else [])
    else:
        mesh = MM.box3d(3, 3, 2, periodic=(True, not wall, True))
    half = 6.0 if D == 2 else 5.0
    vs = dict(dim=D, lo=(-half,) * D, hi=(half,) * D, base=(base,) * D, max_level=levels)
    n = mesh['ncells']
    rng = np.random.default_rng(51 + levels)
    prim = np.concatenate([1 + 0.1 * rng.uniform(-1, 1, (n, 1)), 0.3 * rng.uniform(-1, 1, (n, D)),
                           1 + 0.1 * rng.uniform(-1, 1, (n, 1)), 0.8 + 0.1 * rng.uniform(-1, 1, (n, 1))], axis=1)
    vgas = dict(R=0.5, Pr=0.72, omega=0.74, mu_ref=0.05, T_ref=1.0, model=1)
    cs, dia, o = dia_pair(avs, mesh, vs, vgas, 2e-3, prim, random_tree(vs, 52, 2 if D == 2 else 1, 0.2))
    for _ in range(2):
        dia.step(1)
        o.step(1)
    v, W = dia.get_state()
    assert rel(v, o.phi) < 2e-12 and rel(W, o.W) < 2e-12
    dia.step_implicit(1, 3, 3)
    o.step_implicit(1, 3, 3)
    v, W = dia.get_state()
    assert rel(v, o.phi) < 1e-11 and rel(W, o.W) < 1e-11
    dia.close()
    cs.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [(1279, 1), (40, 32), (43, 30), (11, 13, 9)])
def test_moment_groups(avs, shape, prec):
    """The moments pass on both sides of its grouping by four cells and with
    two and three cells left over: heat fluxes against the same sums in numpy
    over the state read back (FP64 sums of up to 900 terms: 1e-12 of the sum
    of their magnitudes)."""
    D = len(shape)
    mesh = MM.box2d(*shape, periodic=(True, True)) if D == 2 else MM.box3d(*shape)
    vs = dict(dim=D, lo=(-6.0,) * D, hi=(6.0,) * D, base=(8,) * D, max_level=1)
    tree = random_tree(vs, 61, 1, 0.1)
    prim = F.perturbed_uniform(mesh['ncells'], D, 62, amp=0.1, uamp=0.3)
    cs = avs.Case(mesh, vs, GAS, 1e-3, 1.0, prim, precision=prec)
    cs.set_leaves(tree.level, tree.idx)
    q = cs.moments(totals=False)[0].cpu().numpy()[:, D + 2:]
    v, W = cs.get_state()
    v, xi, A = np.asarray(v, dtype=np.float64), tree.centres(), tree.weights()
    c = xi[None] - (W[:, 1:1 + D] / W[:, :1])[:, None]
    e = 0.5 * A * (np.sum(c * c, -1) * v[0] + (v[1] if D == 2 else 0.0))
    ref = np.einsum('ik,ikd->id', e, c)
    assert np.max(np.abs(q - ref)) < 1e-12 * np.max(np.einsum('ik,ikd->id', e, np.abs(c)))
    cs.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_triangles_inner_and_boundary(avs, prec):
    """Cells with three interior faces and with one or two walls: two explicit
    steps (FP64 1e-12 per step; FP32 1e-5 of the field, as the other step
    tests)."""
    mesh = MM.tri_box(5, 4, 71, sides=dict(left=0, right=0, bottom=0, top=0), bcs=[(MM.WALL, (1.0, 0.1, 0.0, 1.1))])
    vs = dict(dim=2, lo=(-6, -6), hi=(6, 6), base=(8, 8), max_level=2)
    prim = F.perturbed_uniform(mesh['ncells'], 2, 72, amp=0.1, uamp=0.3)
    cs, o = make_pair(avs, mesh, vs, GAS, 0.5 * F._cfl_dt(mesh, 0.5, (6.0, 6.0)), prim, tree=random_tree(vs, 73, 2),
                      noise=0.02, seed=74, precision=prec)
    cs.step(2)
    o.step(2)
    v, W = cs.get_state()
    if prec:
        assert fieldrel(W, o.W) < 1e-5 and fieldrel(v, o.phi) < 1e-5
    else:
        assert rel(v, o.phi) < 2e-12 and rel(W, o.W) < 2e-12
