"""Ray batches cut rays into 32 or 16 parts, or walk them whole, by size and
depth; the backward takes records, or walks and keeps them in turns.  All give
the same colours and gradients."""
import numpy as np
import pytest

from paper_2202_08614_amd import _lib, autograd, synth
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu
DEPTH = 4                     # 32 << 4 = 512, 64 << 4 = 1024, 384 << 4 = 6144, 768 << 4 = 12288 rays


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _rays(n, seed, dev):
    import torch
    rng = np.random.default_rng(seed)
    o = np.float32([0.5, 0.5, 0.5]) + 1.5 * _unit(rng, n)
    d = rng.random((n, 3), dtype=np.float32) - o
    t = rng.integers(0, 3, n).astype(np.int32)
    return [torch.from_numpy(np.ascontiguousarray(a, dtype=a.dtype)).to(dev) for a in (o.astype(np.float32), d, t)]


def _unit(rng, n):
    v = rng.standard_normal((n, 3)).astype(np.float32)
    return v / np.linalg.norm(v, axis=1, keepdims=True)


@pytest.mark.parametrize("stop_T", [0.0, 1e-3, 0.3])
@pytest.mark.parametrize("mode", ["f32", "bf16", "fp8", "snap_f32", "snap_bf16"])
def test_ray_batches_of_every_size(dev, mode, stop_T):
    """Against the same rays in a batch that walks them whole: FP32 rounding of
    the parts' products (bound 1e-5), but a ray whose transmittance crosses
    stop_T within rounding may keep or lose what lies behind it."""
    import torch
    dijk = synth.random_tree_leaves(21, DEPTH, p_split=0.8)
    tree = _lib.DeviceTree.from_leaves(dijk, synth.gaussian_coeffs(len(dijk), seed=21), DEPTH, device=dev)
    basis = torch.from_numpy(_lib.time_basis([1.0, 22.2, 47.9])).to(dev)
    kw = dict(stop_T=stop_T, bg=(0.1, 0.2, 0.3))
    if mode.startswith("snap"):
        dt = _lib.FPO_F32 if mode == "snap_f32" else _lib.FPO_BF16
        snap = _lib.bake_times(tree, basis, dt)
        kw.update(snapshot=snap, snapshot_dtype=dt, snapshot_cam_stride=tree.leaf_stride)
    elif mode != "f32":
        tree = _lib.quantize(tree, {"bf16": _lib.FPO_BF16, "fp8": _lib.FPO_FP8_E4M3}[mode])
    opts = _lib.make_opts(**kw)
    o, d, t = _rays(40000, 5, dev)
    note(f"ray batches {mode} stop_T={stop_T}")
    want, want_T = _lib.render_rays(tree, o, d, t, basis, opts, want_T=True)
    for n in (1, 3, 5, 511, 513, 1025, 6145, 12289):
        got, got_T = _lib.render_rays(tree, o[:n].contiguous(), d[:n].contiguous(), t[:n].contiguous(), basis, opts,
                                      want_T=True)
        torch.cuda.synchronize()
        for g, w in ((got, want[:n]), (got_T, want_T[:n])):
            e = (g - w).abs()
            assert float(e.max()) <= 1e-5 + 2 * stop_T
            assert float((e > 1e-5).float().mean()) <= 1e-3


def _grad(tree, rays, basis, g, rgb, opts):
    import torch
    out = torch.zeros_like(tree.coeffs)
    tv = tree.view()
    import ctypes
    o, d, t = rays
    _lib._check(_lib.lib().fpo_render_backward(
        ctypes.byref(tv), *(_lib._t_ptr(a) for a in (o, d, t, basis)), int(basis.shape[0]), int(o.shape[0]),
        ctypes.byref(opts), *(_lib._t_ptr(a) for a in (rgb, g, out)), _lib._stream()))
    return out


@pytest.mark.parametrize("n", [1, 2, 9000])
@pytest.mark.parametrize("stop_T", [0.0, 0.2])
def test_more_records_than_are_staged(dev, n, stop_T):
    """A bar of 256 leaves at depth 8 seen end on: 8 segments in each of 32
    parts, 16 in each of 16 (9000 rays), of which 8 are staged at a time.
    Records, overflowing records (walked again) and the walk without records
    give one gradient, and n copies of the ray n times that of one."""
    import torch
    x = np.arange(256, dtype=np.int32)
    dijk = np.stack([np.full_like(x, 8), x, np.full_like(x, 128), np.full_like(x, 128)], 1)
    k = 0.05 * synth.gaussian_coeffs(256, seed=4)
    k[:, :31] = 0.0                                    # every segment opaque; with stop_T the ray stops inside
    k[:, 0] = 0.18 if stop_T else 0.02
    tree = _lib.DeviceTree.from_leaves(dijk, k, 8, device=dev, sigma_scale=16.0)
    basis = torch.from_numpy(_lib.time_basis([5.0])).to(dev)
    y = np.float32(128.4 / 256)
    o = torch.tensor([[-0.5, y, y]], device=dev).repeat(n, 1).contiguous()
    d = torch.tensor([[1.0, 1e-4, -2e-4]], device=dev).repeat(n, 1).contiguous()
    t = torch.zeros(n, dtype=torch.int32, device=dev)
    g = torch.tensor([[0.3, -0.7, 1.1]], device=dev).repeat(n, 1).contiguous() / n
    rays = (o, d, t)
    plain = _lib.make_opts(stop_T=stop_T)
    note(f"records beyond the stage n={n} stop_T={stop_T}")
    rgb, _ = _lib.render_rays(tree, *rays, basis, plain)
    walked = _grad(tree, rays, basis, g, rgb, plain)
    grads, counts = [], []
    for cap in (512, 100, 1):
        if n * cap > 5_000_000:
            continue
        ws = _lib.record_workspace(n, cap, dev)
        rec = _lib.with_records(plain, ws)
        rgb_r, _ = _lib.render_rays(tree, *rays, basis, rec)
        grads.append(_grad(tree, rays, basis, g, rgb_r, rec))
        counts.append(_lib.record_counts(ws, n).cpu().numpy())
        assert torch.equal(rgb_r, rgb)
    one = _lib.render_rays(tree, *(a[:1].contiguous() for a in rays), basis, plain)[0]
    torch.cuda.synchronize()
    sig = _lib.bake_times(tree, basis)[0, :, 0]
    assert bool((sig > 0).all())
    if n < 9000:
        full = 256 if stop_T == 0.0 else int(counts[0][0])
        assert 100 < full <= 256 and (counts[0] == full).all() and (counts[1] == -1).all()
    assert (counts[-1] == -1).all()
    top = float(walked.abs().max())
    assert top > 0
    # atomics of n equal contributions in any order: n ulps of the sum at most
    for other in grads:
        assert float((other - walked).abs().max()) <= (n + 4) * 2.0 ** -24 * top
    assert float((one - rgb).abs().max()) <= 1e-5


@pytest.mark.parametrize("n", [300, 3000, 40000])
def test_autograd_and_batched_backward_equal_the_direct_call(dev, n):
    """autograd.render keeps records for its backward, _lib.render_backward
    takes large batches through records in pieces: both give fpo_render_backward's
    gradient (parts and whole rays differ by FP32 rounding: 1e-4 of the largest)."""
    import torch
    dijk = synth.random_tree_leaves(22, DEPTH, p_split=0.8)
    tree = _lib.DeviceTree.from_leaves(dijk, synth.gaussian_coeffs(len(dijk), seed=22), DEPTH, device=dev)
    basis = torch.from_numpy(_lib.time_basis([1.0, 22.2, 47.9])).to(dev)
    rays = _rays(n, 6, dev)
    opts = _lib.make_opts(stop_T=1e-3)
    g = torch.randn((n, 3), device=dev, generator=torch.Generator(device=dev).manual_seed(1))
    note(f"backward routes n={n}")
    rgb, _ = _lib.render_rays(tree, *rays, basis, opts)
    direct = _grad(tree, rays, basis, g, rgb, opts)
    batched = _lib.render_backward(tree, *rays, basis, rgb, g, torch.zeros_like(tree.coeffs), opts)
    tree.coeffs.requires_grad_()
    out = autograd.render(tree, *rays, basis, opts)
    (first,) = torch.autograd.grad(out, tree.coeffs, g, retain_graph=True)
    moved = []
    with torch.autograd.graph.saved_tensors_hooks(lambda a: moved.append(1) or a.clone(), lambda a: a.clone()):
        again = autograd.render(tree, *rays, basis, opts)
    (hooked,) = torch.autograd.grad(again, tree.coeffs, g)
    (second,) = torch.autograd.grad(out, tree.coeffs, g)
    torch.cuda.synchronize()
    assert moved and torch.equal(out.detach(), rgb)
    with torch.no_grad():
        quiet = autograd.render(tree, *rays, basis, opts)
    assert not quiet.requires_grad and torch.equal(quiet, rgb)
    top = float(direct.abs().max())
    for other in (batched, first, second, hooked):
        assert float((other - direct).abs().max()) <= 1e-4 * top
