"""fpo_render_backward without records: up to 32 << depth rays in parts, more
with one wave per ray.  Either side of the limit, and past the largest recorded
batch, the gradient is the recorded one up to FP32 rounding: transmittances of
some 30 factors in other orders (30 x 2^-24 each way, in sums over many rays)
stay below 1e-4 of the largest entry."""
import ctypes

import numpy as np
import pytest

from paper_2202_08614_amd import _lib, synth
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu
DEPTH = 4


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _backward(tree, rays, basis, rgb, g, out, opts):
    tv = tree.view()
    _lib._check(_lib.lib().fpo_render_backward(
        ctypes.byref(tv), *(_lib._t_ptr(a) for a in (*rays, basis)), int(basis.shape[0]), int(rays[0].shape[0]),
        ctypes.byref(opts), *(_lib._t_ptr(a) for a in (rgb, g, out)), _lib._stream()))


@pytest.mark.parametrize("stop_T", [0.0, 1e-2])
@pytest.mark.parametrize("n", [1, 63, 32 << DEPTH, (32 << DEPTH) + 1, 2047, 32768, 32771])
def test_walked_gradient_equals_the_recorded_one(dev, n, stop_T):
    import torch
    dijk = synth.random_tree_leaves(23, DEPTH, p_split=0.8)
    tree = _lib.DeviceTree.from_leaves(dijk, synth.gaussian_coeffs(len(dijk), seed=23), DEPTH, device=dev,
                                       sigma_scale=16.0)
    basis = torch.from_numpy(_lib.time_basis([1.0, 22.2, 47.9])).to(dev)
    rng = np.random.default_rng(n)
    v = rng.standard_normal((n, 3))
    o = (0.5 + 1.5 * v / np.linalg.norm(v, axis=1, keepdims=True)).astype(np.float32)
    d = (rng.uniform(0.2, 0.8, (n, 3)) - o).astype(np.float32)
    t = rng.integers(0, 3, n).astype(np.int32)
    rays = [torch.from_numpy(a).to(dev) for a in (o, d, t)]
    g = torch.from_numpy(rng.standard_normal((n, 3)).astype(np.float32)).to(dev)
    plain = _lib.make_opts(stop_T=stop_T)
    note(f"backward n={n} stop_T={stop_T}")
    rgb, _ = _lib.render_rays(tree, *rays, basis, plain)
    got = torch.zeros_like(tree.coeffs)
    _backward(tree, rays, basis, rgb, g, got, plain)
    want = torch.zeros_like(tree.coeffs)
    for a in range(0, n, 32768):
        part = [x[a:a + 32768].contiguous() for x in rays]
        ws = _lib.record_workspace(len(part[0]), 64, dev)
        rec = _lib.with_records(plain, ws)
        rgb_a, _ = _lib.render_rays(tree, *part, basis, rec)
        _backward(tree, part, basis, rgb_a, g[a:a + 32768].contiguous(), want, rec)
    lib = _lib.render_backward(tree, *rays, basis, rgb, g, torch.zeros_like(tree.coeffs), plain)
    torch.cuda.synchronize()
    top = float(want.abs().max())
    assert top > 0
    assert float((got - want).abs().max()) <= 1e-4 * top
    assert float((lib - want).abs().max()) <= 1e-4 * top
