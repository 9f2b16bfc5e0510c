"""Which tiles go out in which order, on which XCD: single rows for cameras that
read the same records, bands of rows for 8 and 16 cameras with records of their
own and for views from nearby, whole rays in launches that see many pixels of
the scene.  Every camera's image is the one it has alone (FP32 rounding of the
parts that small launches cut rays into, 1e-5; no early stop)."""
import numpy as np
import pytest

from paper_2202_08614_amd import _lib, synth
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu
DEPTH = 3                # whole rays from 1024 << 3 pixels that see the leaves, 256 << 3 from nearby


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.mark.parametrize("dtype", [_lib.FPO_F32, _lib.FPO_BF16])
@pytest.mark.parametrize("own", [True, False])
@pytest.mark.parametrize("n,w,h", [(1, 150, 141), (7, 33, 17), (8, 97, 61), (9, 97, 61), (16, 101, 67), (19, 64, 49)])
@pytest.mark.parametrize("radius", [1.5, 0.1])
def test_cameras_of_one_launch(dev, dtype, own, n, w, h, radius):
    import torch
    dijk = synth.random_tree_leaves(61, DEPTH, p_split=0.85)
    tree = _lib.DeviceTree.from_leaves(dijk, synth.gaussian_coeffs(len(dijk), seed=61), DEPTH, device=dev,
                                       sigma_scale=8.0)
    times = np.linspace(1.0, 50.0, n)
    cams = [synth.ring_camera(0.7 * i, 0.3 - 0.03 * i, radius, 50.0, w, h, float(t)) for i, t in enumerate(times)]
    snaps = _lib.bake_times(tree, torch.from_numpy(_lib.time_basis(times)).to(dev), dtype)
    stride = tree.leaf_stride if own else 0
    note(f"tile order n={n} {w}x{h} own={own} radius={radius}")
    kw = dict(bg=(0.1, 0.2, 0.3), snapshot_dtype=dtype)
    got, T = _lib.render(tree, cams, _lib.make_opts(snapshot=snaps, snapshot_cam_stride=stride, **kw), want_T=True)
    for i, cam in enumerate(cams):
        one, one_T = _lib.render(tree, [cam], _lib.make_opts(snapshot=snaps[i if own else 0], **kw), want_T=True)
        torch.cuda.synchronize()
        assert float((got[i] - one[0]).abs().max()) <= 1e-5 and float((T[i] - one_T[0]).abs().max()) <= 1e-5
    assert float(T.min()) < 0.9
