"""Kernel variants at the sizes where their dispatch or their tiling can go
wrong, against the FP64 oracle on identical seeded inputs."""
import numpy as np
import pytest

from workloads import fields as F
from workloads import meshes as MM

from test_gpu_implicit import dia_pair
from test_gpu_parity import make_pair, random_tree, rel

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
