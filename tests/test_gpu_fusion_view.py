"""fpo_fusion_view (observations in lists per leaf) against fpo_fusion_observe
and fpo_fusion_apply."""
import ctypes

import numpy as np
import pytest

from paper_2202_08614_amd import _lib, synth
from paper_2202_08614_amd.fusion import Fusion
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _scene(dev, depth, seed, clip=True, dense=1.0):
    import torch
    dijk = synth.random_tree_leaves(seed, depth, p_split=0.7)          # mixed depths
    tree = _lib.DeviceTree.from_leaves(dijk, np.zeros((len(dijk), 166), np.float32), depth, device=dev, clip=clip,
                                       leaf_stride=len(dijk) + 3)
    g = torch.Generator(device=dev).manual_seed(seed)
    n = tree.leaf_stride
    values = dense * torch.randn((n, 32), generator=g, device=dev)
    values[:, 28:] = 0.0
    count = torch.randint(0, 5, (n,), generator=g, device=dev, dtype=torch.int32)
    weight = torch.rand((n,), generator=g, device=dev) * (count > 0)
    rng = np.random.default_rng(seed)
    field = synth.Field(mu=rng.uniform(0.3, 0.7, (8, 3)), w=rng.uniform(0.05, 0.2, 8), a=rng.uniform(0.2, 1.0, 8),
                        u=rng.normal(0.0, 2.0, (3, 3)), v=rng.normal(0.0, 1.0, (3, 3)), b=rng.normal(0.0, 0.5, 3))
    return tree, values, weight, count, field


def _check(f, values, weight, count, tie):
    """The same terms in another order, and transmittances composed of parts:
    1e-5 relative to the values' scale; `tie` leaves may differ where a
    segment's transmittance meets tau within rounding."""
    off = ((f.values - values).abs() > 1e-5 * (1.0 + values.abs())).any(1)
    off |= (f.weight - weight).abs() > 1e-5
    off |= f.count != count
    assert int(off.sum()) <= tie, int(off.sum())


@pytest.mark.parametrize("depth,w,h", [(5, 1, 1), (5, 3, 5), (6, 37, 23), (6, 181, 182), (6, 210, 170), (4, 400, 301)])
@pytest.mark.parametrize("dense", [0.3, 8.0])
def test_view_equals_observe_and_apply(dev, depth, w, h, dense):
    """16 lanes a ray up to 512 << depth pixels (181 x 182 is past it at depth
    6), 8 above; views from outside and from inside the leaves' box."""
    import torch
    tree, values, weight, count, field = _scene(dev, depth, 30 + depth, clip=w % 2 == 1, dense=dense)
    f = Fusion(tree, values.clone(), field, weight=weight.clone(), count=count.clone())
    acc = torch.zeros_like(f.acc)
    for j in range(3):
        cam = synth.ring_camera(0.9 * j, 0.3, 0.2 if j == 1 else 1.5, 60.0, w, h, 0.0)
        note(f"fusion view depth={depth} {w}x{h} view {j}")
        v, wt, c = f.values.clone(), f.weight.clone(), f.count.clone()
        _lib.fusion_observe(tree, v, cam, field, acc, f.tau)
        _lib.fusion_apply(v, wt, c, acc, tree.n_leaves)
        f.view(cam)
        torch.cuda.synchronize()
        _check(f, v, wt, c, tie=2)
        assert not bool(f.acc.any())


def test_view_takes_earlier_observations_and_small_workspaces(dev):
    """What earlier observe calls left in acc is part of the update; a workspace
    that cannot hold the observations gives the same update; one below the
    lists' heads is refused."""
    import torch
    tree, values, weight, count, field = _scene(dev, 6, 44)
    cams = [synth.ring_camera(0.5 * j, 0.2, 1.5, 50.0, 160, 120, 0.0) for j in range(2)]
    fs = _lib.field_struct(field)
    acc = torch.zeros((tree.leaf_stride, 32), device=dev)
    _lib.fusion_observe(tree, values, cams[0], fs, acc)
    want = [values.clone(), weight.clone(), count.clone(), acc.clone()]
    _lib.fusion_observe(tree, want[0], cams[1], fs, want[3])
    _lib.fusion_apply(*want, tree.n_leaves)
    tv, cs = tree.view(), _lib.camera_struct([cams[1]])
    full = _lib.lib().fpo_fusion_view_bytes(ctypes.byref(tv), cs)
    heads = 256 * 40 + tree.n_leaves * 4 + 160 * 120 * 16 * 4 + 4096
    assert 0 < heads < full
    for nbytes in (full, heads, heads + 20 * 64 * 300, 4096):
        got = [values.clone(), weight.clone(), count.clone(), acc.clone()]
        ws = torch.full((nbytes + 256,), 171, dtype=torch.uint8, device=dev)
        note(f"fusion view workspace {nbytes}")
        st = _lib.lib().fpo_fusion_view(ctypes.byref(tv), *(_lib._t_ptr(a) for a in got[:3]), cs, ctypes.byref(fs),
                                        1e-3, _lib._t_ptr(got[3]), _lib._t_ptr(ws), nbytes, _lib._stream())
        torch.cuda.synchronize()
        assert bool((ws[nbytes:] == 171).all())
        if nbytes == 4096:
            assert st == 1 and all(torch.equal(a, b) for a, b in zip(got, (values, weight, count, acc)))
            continue
        assert st == 0
        assert torch.equal(got[2], want[2])
        for a, b in zip(got[:2], want[:2]):
            assert bool(((a - b).abs() <= 1e-5 * (1.0 + b.abs())).all())
        assert not bool(got[3].any())


def test_view_under_capture_takes_the_atomic_sums(dev):
    import torch
    tree, values, weight, count, field = _scene(dev, 5, 45)
    cam = synth.ring_camera(0.4, 0.2, 1.5, 50.0, 64, 48, 0.0)
    f = Fusion(tree, values.clone(), field, weight=weight.clone(), count=count.clone())
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        f.view(cam)
    for _ in range(3):
        v, wt, c = f.values.clone(), f.weight.clone(), f.count.clone()
        acc = torch.zeros_like(f.acc)
        _lib.fusion_observe(tree, v, cam, field, acc, f.tau)
        _lib.fusion_apply(v, wt, c, acc, tree.n_leaves)
        g.replay()
        torch.cuda.synchronize()
        _check(f, v, wt, c, tie=0)
