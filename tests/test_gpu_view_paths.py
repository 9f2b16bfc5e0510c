"""Camera renders take several routes by size: lanes of one ray sharing its
chord (small launches), rows or bands of tiles per XCD, and decoding the leaves
at the cameras' times first (views large against the tree).  The routes give
the same images."""
import ctypes
import math

import numpy as np
import pytest

from paper_2202_08614_amd import _lib, synth
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _tree(dev, seed=5, depth=6, stride_pad=0, k=None):
    dijk = synth.random_tree_leaves(seed, depth, p_split=0.7)          # mixed depths
    k = synth.gaussian_coeffs(len(dijk), seed=seed) if k is None else k(len(dijk))
    return _lib.DeviceTree.from_leaves(dijk, k, depth, device=dev, leaf_stride=len(dijk) + stride_pad)


def _close(a, b, stop_T):
    """Composing a chord from parts and summing a leaf's terms in another order
    move a colour by FP32 rounding: the parity bar 1e-4 bounds sums of 31 terms
    (31 * 2^-23 * sum |k b| < 5e-5 in optical depth).  A ray whose
    transmittance crosses stop_T within rounding may keep or lose what lies
    behind it (at most stop_T)."""
    d = (a - b).abs()
    assert float(d.max()) <= 1e-4 + 2 * stop_T, float(d.max())
    assert float((d > 1e-4).float().mean()) <= 1e-3


@pytest.mark.parametrize("stop_T", [0.0, 1e-3, 0.3])
@pytest.mark.parametrize("mode", ["f32", "bf16", "fp8", "snap_f32", "snap_bf16"])
def test_lanes_per_ray_and_rows(dev, mode, stop_T):
    """One camera alone (16 lanes a ray), and copies of it that fill a launch
    past each limit (8 lanes, one lane; rows of tiles, and a band per XCD for 8
    and 16 copies)."""
    import torch
    tree = _tree(dev)
    t = 17.3
    kw = dict(stop_T=stop_T, bg=(0.2, 0.4, 0.1))
    if mode.startswith("snap"):
        dt = _lib.FPO_F32 if mode == "snap_f32" else _lib.FPO_BF16
        basis = torch.from_numpy(_lib.time_basis([t])).to(dev)
        snap = _lib.bake_times(tree, basis, dt)
        kw.update(snapshot=snap, snapshot_dtype=dt)
    elif mode != "f32":
        tree = _lib.quantize(tree, {"bf16": _lib.FPO_BF16, "fp8": _lib.FPO_FP8_E4M3}[mode])
    opts = _lib.make_opts(**kw)
    for w, h in ((1, 1), (3, 5), (101, 67)):
        cam = synth.ring_camera(0.7, 0.3, 1.5, 40.0, w, h, t)
        note(f"lanes per ray {mode} {w}x{h}")
        want, want_T = _c_render(tree, [cam] * 1, opts, dev)
        many = [cam] * (16 if w < 100 else 80)
        got, got_T = _c_render(tree, many, opts, dev)
        torch.cuda.synchronize()
        for j in (0, 7, len(many) - 1):
            _close(got[j], want[0], stop_T)
            _close(got_T[j], want_T[0], stop_T)
        nine, _ = _c_render(tree, [cam] * 9, opts, dev)
        _close(nine[8], want[0], stop_T)


def _c_render(tree, cams, opts, dev):
    """fpo_render itself (no decode)."""
    import torch
    n, H, W = len(cams), cams[0].height, cams[0].width
    rgb = torch.full((n, H, W, 3), float("nan"), device=dev)
    T = torch.full((n, H, W), float("nan"), device=dev)
    tv = tree.view()
    _lib._check(_lib.lib().fpo_render(ctypes.byref(tv), _lib.camera_struct(cams), n, ctypes.byref(opts),
                                      _lib._t_ptr(rgb), _lib._t_ptr(T), _lib._stream()))
    return rgb, T


def _c_decoded(tree, cams, opts, dev, n_times):
    import torch
    n, H, W = len(cams), cams[0].height, cams[0].width
    rgb = torch.full((n, H, W, 3), float("nan"), device=dev)
    T = torch.full((n, H, W), float("nan"), device=dev)
    nbytes = 2048 + n_times * tree.n_leaves * 128
    ws = torch.full((nbytes + 256,), 255, dtype=torch.uint8, device=dev)
    tv = tree.view()
    _lib._check(_lib.lib().fpo_render_decoded(ctypes.byref(tv), _lib.camera_struct(cams), n, ctypes.byref(opts),
                                              _lib._t_ptr(rgb), _lib._t_ptr(T), _lib._t_ptr(ws), nbytes,
                                              _lib._stream()))
    torch.cuda.synchronize()
    assert bool((ws[nbytes:] == 255).all())          # nothing written past the workspace it was given
    return rgb, T


@pytest.mark.parametrize("store", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("n_cams,n_t,fit", [(1, 1, 1), (3, 3, 3), (5, 5, 2), (20, 18, 16), (20, 1, 1), (18, 4, 16)])
def test_decoded_equals_direct(dev, store, n_cams, n_t, fit):
    tree = _tree(dev, seed=8, stride_pad=3)
    if store != "f32":
        tree = _lib.quantize(tree, {"bf16": _lib.FPO_BF16, "fp8": _lib.FPO_FP8_E4M3}[store])
    cams = [synth.ring_camera(0.3 * j, 0.2, 1.5, 45.0, 37, 23, 60.0 * ((j * 7) % n_t) / n_t + 0.4)
            for j in range(n_cams)]
    for stop_T in (0.0, 1e-3):
        opts = _lib.make_opts(stop_T=stop_T, bg=(0.1, 0.0, 0.3))
        note(f"decoded {store} {n_cams} cameras {n_t} times, {fit} fit")
        want, want_T = _c_render(tree, cams, opts, dev)
        got, got_T = _c_decoded(tree, cams, opts, dev, fit)
        _close(got, want, stop_T)
        _close(got_T, want_T, stop_T)


def test_decoded_takes_infinite_coefficients_as_the_direct_render(dev):
    """An infinite SH coefficient next to the density ones, an infinite and a
    NaN density coefficient: the same pixels are finite, and equal."""
    import torch

    def coeffs(n):
        k = synth.gaussian_coeffs(n, seed=3)
        k[::7, 31] = np.inf
        k[3::11, 0] = np.inf
        k[5::13, 2] = np.nan
        return k
    tree = _tree(dev, k=coeffs)
    cams = [synth.ring_camera(0.4 * j, 0.2, 1.5, 45.0, 40, 30, 3.0 + 7.0 * j) for j in range(4)]
    opts = _lib.make_opts()
    for fit in (1, 4):
        want, want_T = _c_render(tree, cams, opts, dev)
        got, got_T = _c_decoded(tree, cams, opts, dev, fit)
        torch.cuda.synchronize()
        assert torch.equal(torch.isfinite(want), torch.isfinite(got))
        m = torch.isfinite(want)
        assert float((want[m] - got[m]).abs().max()) <= 1e-4


def test_decode_is_chosen_by_size_and_refused_where_unsupported(dev):
    """fpo_render_decode_bytes: 0 for small views, snapshots, skip flags and
    other layouts; the records of the distinct times else.  render() takes the
    decoded route and equals the direct one, and under capture the direct one."""
    import torch
    tree = _tree(dev, depth=7, seed=11)
    L = _lib.lib()

    def need(cams, **kw):
        tv = kw.pop("view", None) or tree.view()
        o = _lib.make_opts(**kw)
        return L.fpo_render_decode_bytes(ctypes.byref(tv), _lib.camera_struct(cams), len(cams), ctypes.byref(o))
    small = [synth.ring_camera(0.1, 0.2, 1.5, 45.0, 16, 16, 1.0)]
    big = [synth.ring_camera(0.1 + j, 0.2, 1.5, 45.0, 1920, 1080, 1.0 + j // 2) for j in range(4)]
    assert need(small) == 0
    assert need(big) == 2048 + 2 * tree.n_leaves * 128
    snap = torch.zeros((tree.leaf_stride, 32), device=dev)
    assert need(big, snapshot=snap) == 0
    bits = torch.zeros(8192, dtype=torch.int32, device=dev)
    ws = _lib.skip_workspace(4, 1080, 1920, dev)
    assert need(big, flags=_lib.FPO_RENDER_SKIP_COARSE, coarse_bits=bits, workspace=ws) == 0
    other = tree.view()
    other.layout = _lib.make_layout(n_sigma=11)
    assert need(big, view=other) == 0
    opts = _lib.make_opts(stop_T=1e-3)
    direct, direct_T = _c_render(tree, big, opts, dev)
    rgb, T = _lib.render(tree, big, opts, want_T=True)
    _close(rgb, direct, 1e-3)
    _close(T, direct_T, 1e-3)
    out = torch.empty_like(rgb)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _lib.render(tree, big, opts, rgb=out)
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, direct)
    with pytest.raises(_lib.FpoError):
        _c_decoded(tree, small, _lib.make_opts(snapshot=snap), dev, 1)
    with pytest.raises(_lib.FpoError):
        _c_decoded(tree, small, _lib.make_opts(), dev, 0)
