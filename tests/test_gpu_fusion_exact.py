"""Fusion.view observes exactly the segments that fpo_fusion_observe does, once
each: the same leaves are counted, and values and weights differ by the order
of a leaf's sums only.  A leaf may get an observation from every pixel; the
roundings (2^-24 each) of n sums of values below 10, taken in two orders, move
their mean by 10 sqrt(n) 2^-24 and no leaf is exempt."""
import numpy as np
import pytest

from paper_2202_08614_amd import _lib, synth
from paper_2202_08614_amd.fusion import Fusion
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _full(depth, keep):
    """The cells of the finest lattice that keep(x, y, z) selects."""
    g = 1 << depth
    x, y, z = np.meshgrid(*(np.arange(g, dtype=np.int32),) * 3, indexing="ij")
    sel = keep(x, y, z)
    return np.stack([np.full(int(sel.sum()), depth, np.int32), x[sel], y[sel], z[sel]], 1)


def _camera(eye, fwd, fov, w, h):
    return synth.Camera(eye=eye, fwd=fwd, up=(0.0, 1.0, 0.0) if abs(fwd[1]) < 0.9 else (1.0, 0.0, 0.0),
                        fov_y_deg=fov, width=w, height=h, time=0.0)


def _compare(dev, dijk, depth, cams, density, tau, clip=True, sigma_scale=64.0):
    import torch
    tree = _lib.DeviceTree.from_leaves(dijk, np.zeros((len(dijk), 166), np.float32), depth, device=dev, clip=clip,
                                       sigma_scale=sigma_scale)
    gen = torch.Generator(device=dev).manual_seed(len(dijk))
    n = tree.leaf_stride
    values = torch.randn((n, 32), generator=gen, device=dev)
    values[:, 0] *= density
    values[:, 28:] = 0.0
    count = torch.randint(0, 5, (n,), generator=gen, device=dev, dtype=torch.int32)
    weight = torch.rand((n,), generator=gen, device=dev) * (count > 0)
    field = synth.fusion_field()
    f = Fusion(tree, values, field, tau=tau, weight=weight, count=count)
    acc = torch.zeros_like(f.acc)
    seen = 0
    for i, cam in enumerate(cams):
        note(f"fusion exact depth={depth} leaves={len(dijk)} {cam.width}x{cam.height} view {i}")
        v, wt, c = f.values.clone(), f.weight.clone(), f.count.clone()
        before = f.count.clone()
        _lib.fusion_observe(tree, v, cam, field, acc, tau)
        _lib.fusion_apply(v, wt, c, acc, tree.n_leaves)
        f.view(cam)
        torch.cuda.synchronize()
        assert torch.equal(f.count, c), int((f.count != c).sum())
        for a, b in ((f.values, v), (f.weight, wt)):
            off = (a - b).abs() > 10.0 * (cam.width * cam.height) ** 0.5 * 2.0 ** -24 * (1.0 + b.abs())
            assert not bool(off.any()), (i, int(off.sum()), float((a - b).abs().max()))
        seen += int((c != before).sum())
    return seen


@pytest.mark.parametrize("w,h", [(160, 120), (400, 300)])
@pytest.mark.parametrize("clip", [True, False])
def test_leaves_at_a_face_seen_along_it(dev, w, h, clip):
    """Cameras just outside a face's plane, looking along it and at grazing
    angles, with a leaf in every cell of the cube's outer layer; no densities,
    so that every segment counts with T = 1."""
    dijk = _full(5, lambda x, y, z: (np.minimum(np.minimum(x, y), z) == 0) | (np.maximum(np.maximum(x, y), z) == 31))
    cams = [_camera((-0.003, 0.5, 2.0), (0.0, 0.0, -1.0), 40.0, w, h),
            _camera((0.5, 1.002, 2.1), (0.0, -0.001, -1.0), 40.0, w, h),
            _camera((0.5, 0.5, 1.0), (0.3, 0.1, -1.0), 60.0, w, h),           # the eye on a face
            _camera((-0.3, 1.0004, 1.3), (1.0, -0.05, -0.9), 50.0, w, h),     # across an edge
            synth.ring_camera(0.7, 0.26, 1.6, 40.0, w, h, 0.0)]
    assert _compare(dev, dijk, 5, cams, 0.0, 1e-30, clip=clip) > 2000


@pytest.mark.parametrize("tau", [1e-3, 0.2])
def test_segments_whose_transmittance_meets_tau(dev, tau):
    """A solid ball of random densities, in which most rays end: the segments
    on either side of tau are those of fpo_fusion_observe."""
    dijk = _full(6, lambda x, y, z: (x - 31.5) ** 2 + (y - 31.5) ** 2 + (z - 31.5) ** 2 < 28.0 ** 2)
    cams = [synth.ring_camera(0.4 * j, 0.3 - 0.05 * j, 1.5, 45.0, 500, 460, 0.0) for j in range(12)]
    assert _compare(dev, dijk, 6, cams, 1.0, tau) > 20000


@pytest.mark.parametrize("w,h", [(1, 1), (64, 1), (7, 9), (65, 33), (700, 500)])
def test_mixed_depths_and_ragged_images(dev, w, h):
    dijk = synth.random_tree_leaves(71, 7, p_split=0.72)
    cams = [synth.ring_camera(0.9 * j, 0.3, 0.2 if j == 1 else 1.5, 50.0, w, h, 0.0) for j in range(4)]
    _compare(dev, dijk, 7, cams, 0.5, 1e-3)
