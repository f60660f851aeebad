"""Every form of the target, the interface stage and pass C, alone against the
FP64 oracle and batched against the cases alone, bit for bit.  The sizes are
held to the forms they are here for."""
import numpy as np
import pytest

from workloads import fields as F
from workloads import meshes as MM

import forms
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

# name: (mesh shape, base, levels, fraction of roots split, target, interface
# stage, one wave per cell); target and interface stage "group" for the
# workgroup form, else the lanes with one share or several
SIZES = {
    # the largest tables that the lanes take (144 KiB), and the first beyond
    "limit_2d_fp64": ((33, 33), 9, 3, 0.05, "one", "one", True),
    "limit_2d_fp32": ((37, 36), 9, 4, 0.05, "one", "one", False),
    "limit_3d_fp64": ((8, 8, 9), 6, 3, 0.02, "one", "one", False),
    "limit_3d_fp32": ((9, 9, 11), 6, 4, 0.02, "one", "one", False),
    "beyond_2d_fp64": ((33, 33), 73, 0, 0.0, "group", "group", False),
    # one lane short of a group of 64 cells, exactly one, one cell in the second
    "cells_63": ((9, 7), 5, 1, 0.3, "one", "group", False),
    "cells_64": ((8, 8), 5, 1, 0.3, "one", "group", False),
    "cells_65": ((13, 5), 5, 1, 0.3, "one", "group", False),
    # split leaves
    "split_2d": ((35, 31), 32, 0, 0.0, "several", "several", False),
    "split_target_2d": ((20, 21), 20, 0, 0.0, "several", "group", False),
    "split_3d": ((9, 9, 9), 11, 0, 0.0, "several", "several", False),
    # pass C with one wave per cell: fewer leaves than lanes, one leaf per
    # lane, and two rounds of both load schemes
    "wave_2d": ((27, 28), 5, 1, 0.3, "one", "one", True),
    "wave_64_2d": ((27, 28), 8, 0, 0.0, "one", "one", True),
    "wave_3_2d": ((45, 45), 8, 1, 0.7, "one", "one", True),
    "wave_3d": ((8, 8, 9), 4, 0, 0.0, "one", "one", True),
    "small_2d": ((5, 4), 16, 0, 0.0, "group", "group", False),
    "small_3d": ((3, 3, 2), 6, 1, 0.2, "group", "group", False),
}


def build(name, prec):
    shape, base, levels, p, *want = SIZES[name]
    D = len(shape)
    if D == 2:
        mesh = MM.box2d(*shape, periodic=(True, False), sides=dict(bottom=0, top=0),
                        bcs=[(MM.WALL, (1.0, 0.1, 0.0, 1.1))])
    else:
        mesh = MM.box3d(*shape)
    half = 6.0 if D == 2 else 5.0
    vs = dict(dim=D, lo=(-half,) * D, hi=(half,) * D, base=(base,) * D, max_level=levels)
    tree = random_tree(vs, 22, 1 if levels else 0, p)
    prim = F.perturbed_uniform(mesh['ncells'], D, 21, amp=0.1, uamp=0.3)
    numax = 2 * base * 2 ** levels
    kind = lambda s: "group" if s == 0 else "one" if s == 1 else "several"  # noqa: E731
    got = [kind(forms.shares(D, prec, mesh['ncells'], tree.n, numax, 0)),
           kind(forms.shares(D, prec, mesh['nfaces'], tree.n, numax, 1)), forms.wave(D, prec, mesh['ncells'], tree.n, numax)]
    assert got == want, (name, prec, tree.n, got)
    return mesh, vs, 0.5 * F._cfl_dt(mesh, 1.0, (half,) * D), prim, tree


ALONE = [
    ("cells_63", 0), ("cells_64", 0), ("cells_65", 0),
    ("limit_2d_fp64", 0), ("limit_2d_fp32", 1), ("limit_3d_fp64", 0), ("limit_3d_fp32", 1), ("beyond_2d_fp64", 0),
    ("split_2d", 0), ("split_2d", 1), ("split_target_2d", 0), ("split_3d", 0), ("split_3d", 1),
    ("wave_2d", 0), ("wave_2d", 1), ("wave_64_2d", 0), ("wave_3_2d", 0), ("wave_3_2d", 1), ("wave_3d", 0), ("wave_3d", 1)]
# members in different forms, so that every launch of a stage holds some of them
BATCHED = [
    (("split_2d", "small_2d", "wave_2d", "split_target_2d"), 0),
    (("split_2d", "small_2d", "wave_2d", "split_target_2d"), 1),
    (("small_2d", "wave_64_2d", "limit_2d_fp64", "beyond_2d_fp64"), 0),
    (("split_3d", "small_3d", "wave_3d"), 0),
    (("small_3d", "split_3d", "wave_3d"), 1),
]


@pytest.mark.parametrize("name,prec", ALONE)
def test_forms_match_the_oracle(avs, name, prec):
    """One explicit step (FP64 1e-12, FP32 1e-5 of the field, as the other
    step tests)."""
    mesh, vs, dt, prim, tree = build(name, prec)
    cs, o = make_pair(avs, mesh, vs, GAS, dt, prim, tree=tree, noise=0.02, seed=23, precision=prec, cap=tree.n)
    cs.step(1)
    o.step(1)
    v, W = cs.get_state()
    if prec:
        assert fieldrel(W, o.W) < 1e-5 and fieldrel(v, o.phi) < 1e-5
    else:
        assert rel(v, o.phi) < 1e-12 and rel(W, o.W) < 1e-12
    cs.close()


@pytest.mark.parametrize("names,prec", BATCHED)
def test_batched_forms_equal_the_cases_alone(avs, names, prec):
    """Three steps eagerly (both orientations of the state's buffers), then by
    graph, bit for bit."""
    import torch
    stream = torch.cuda.Stream()

    def cases():
        out = []
        for name in names:
            mesh, vs, dt, prim, tree = build(name, prec)
            cs = avs.Case(mesh, vs, GAS, dt, 1.0, prim, precision=prec, stream=stream, leaf_capacity=tree.n)
            cs.set_leaves(tree.level, tree.idx)
            out.append(cs)
        return out
    with torch.cuda.stream(stream):
        solo, grouped = cases(), cases()
        batch = avs.Batch(grouped)
        for n, graph in ((3, False), (3, True), (2, True), (3, True)):
            for cs in solo:
                cs.step(n)
            batch.step(n, graph=graph)
            batch.check()
            for a, b in zip(solo, grouped):
                va, Wa = a.get_state()
                vb, Wb = b.get_state()
                assert np.array_equal(va, vb) and np.array_equal(Wa, Wb)
        batch.close()
        for cs in solo + grouped:
            cs.close()
