"""Rays cut into parts meet every segment exactly once.  In a cube full of
leaves of one constant density the transmittance of any ray is
exp(-sigma * chord), whatever its segments are, so a segment that two parts
report, or none, shows.  Bound: up to 200 segments, each with a rounded length,
exponential and product (3 x 2^-24), and a chord known to a few 2^-23 in a
medium of optical depth at most 3.5: 5e-5.  One cell of the lattice along a ray
is worth 3e-2."""
import numpy as np
import pytest

from paper_2202_08614_amd import _lib, synth
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu
DEPTH = 5                     # ray batches: 32 parts up to 2048 rays (F32: 1024), 16 up to 12288 and more, then whole
SIGMA = 2.0


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.fixture(scope="module")
def full(dev):
    g = 1 << DEPTH
    x, y, z = (a.reshape(-1).astype(np.int32) for a in np.meshgrid(*(np.arange(g),) * 3, indexing="ij"))
    dijk = np.stack([np.full_like(x, DEPTH), x, y, z], 1)
    k = np.zeros((len(dijk), 166), np.float32)
    k[:, 0] = SIGMA / 64.0                    # constant over time
    return _lib.DeviceTree.from_leaves(dijk, k, DEPTH, device=dev, sigma_scale=64.0)


def _chord(o, d):
    o, d = o.astype(np.float64), d.astype(np.float64)
    d = d / np.linalg.norm(d, axis=1, keepdims=True)
    with np.errstate(divide="ignore", invalid="ignore"):
        a, b = (0.0 - o) / d, (1.0 - o) / d
    lo = np.maximum(np.nanmax(np.minimum(a, b), 1), 0.0)
    hi = np.nanmin(np.maximum(a, b), 1)
    return np.maximum(hi - lo, 0.0)


def _along_planes(n, seed):
    """Rays that run almost along one or two planes of the lattice and start
    within a few roundings of them, on either side, along any axis."""
    rng = np.random.default_rng(seed)
    o = np.empty((n, 3), np.float32)
    d = np.empty((n, 3), np.float32)
    plane = rng.integers(1, 1 << DEPTH, (n, 2)).astype(np.float32) / (1 << DEPTH)
    steps = rng.integers(-6, 7, (n, 2))
    for c in range(2):
        v = plane[:, c]
        for s in range(1, 7):
            v = np.where(steps[:, c] >= s, np.nextafter(v, np.float32(2)), v)
            v = np.where(steps[:, c] <= -s, np.nextafter(v, np.float32(-1)), v)
        o[:, c] = v
        tiny = rng.choice([-1.0, 1.0], n) * 10.0 ** rng.uniform(-9.0, -4.0, n)
        d[:, c] = np.where(rng.random(n) < 0.3, rng.uniform(-0.4, 0.4, n), tiny)
    back = rng.random(n) < 0.5
    o[:, 2] = np.where(back, 1.001, -0.001)
    d[:, 2] = np.where(back, -1.0, 1.0)
    for r in range(3):                        # every axis in turn
        at = np.arange(n) % 3 == r
        o[at], d[at] = np.roll(o[at], r, 1), np.roll(d[at], r, 1)
    return o, d


def _across(n, seed):
    rng = np.random.default_rng(seed)
    v = rng.standard_normal((n, 3))
    o = (0.5 + 1.5 * v / np.linalg.norm(v, axis=1, keepdims=True)).astype(np.float32)
    return o, (rng.uniform(0.1, 0.9, (n, 3)) - o).astype(np.float32)


def _opts(mode, tree, basis):
    """Options, and the snapshot that they point to."""
    if mode == "f32":
        return _lib.make_opts(), None
    dt = _lib.FPO_F32 if mode == "snap_f32" else _lib.FPO_BF16
    snap = _lib.bake_times(tree, basis, dt)
    return _lib.make_opts(snapshot=snap, snapshot_dtype=dt), snap


@pytest.mark.parametrize("kind", [_along_planes, _across])
@pytest.mark.parametrize("n", [1000, 1500, 9000, 60000])
@pytest.mark.parametrize("mode", ["f32", "snap_f32"])
def test_transmittance_of_a_uniform_medium(dev, full, kind, n, mode):
    import torch
    basis = torch.from_numpy(_lib.time_basis([7.0])).to(dev)
    o, d = kind(n, 11 + n)
    opts, _keep = _opts(mode, full, basis)
    note(f"uniform medium {kind.__name__} {mode} n={n}")
    _, T = _lib.render_rays(full, torch.from_numpy(o).to(dev), torch.from_numpy(d).to(dev),
                            torch.zeros(n, dtype=torch.int32, device=dev), basis, opts, want_T=True)
    torch.cuda.synchronize()
    err = np.abs(T.cpu().numpy().astype(np.float64) - np.exp(-SIGMA * _chord(o, d)))
    assert err.max() <= 5e-5, (int((err > 5e-5).sum()), err.max(), o[err.argmax()], d[err.argmax()])


def test_a_ray_one_rounding_below_a_plane(dev):
    """Two columns of cells beside the plane x = 1/4, of which only the lower one
    is dense.  A ray that starts one rounding below the plane and reaches it at
    0.45 is in the dense column until then, also where x + t d rounds onto the
    plane from 0.22 on."""
    import torch
    z = np.arange(32, dtype=np.int32)
    dijk = np.concatenate([np.stack([np.full_like(z, DEPTH), np.full_like(z, x), np.full_like(z, 16), z], 1)
                           for x in (7, 8)])
    k = np.zeros((64, 166), np.float32)
    k[:32, 0] = SIGMA / 64.0
    tree = _lib.DeviceTree.from_leaves(dijk, k, DEPTH, device=dev, sigma_scale=64.0)
    basis = torch.from_numpy(_lib.time_basis([7.0])).to(dev)
    x0 = np.nextafter(np.float32(0.25), np.float32(0))
    step = np.float32((0.25 - float(x0)) / 0.45)
    for n in (1, 4000, 20000):
        o = torch.tensor([[float(x0), 16.5 / 32, 0.0]], device=dev).repeat(n, 1).contiguous()
        d = torch.tensor([[float(step), 0.0, 1.0]], device=dev).repeat(n, 1).contiguous()
        note(f"one rounding below a plane n={n}")
        _, T = _lib.render_rays(tree, o, d, torch.zeros(n, dtype=torch.int32, device=dev), basis, _lib.make_opts(),
                                want_T=True)
        torch.cuda.synchronize()
        assert float((T - float(np.exp(-SIGMA * 0.45))).abs().max()) <= 1e-4, float(T[0])


@pytest.mark.parametrize("mode,w,h", [("f32", 60, 50), ("snap_f32", 60, 50), ("snap_f32", 200, 300),
                                      ("snap_bf16", 200, 300), ("snap_f32", 500, 400)])
def test_cameras_along_the_axes(dev, full, mode, w, h):
    """Camera renders with 16 and 8 lanes a ray and with one: eyes on planes of
    the lattice and a rounding beside them, looking along an axis."""
    import torch
    import oracle
    basis = torch.from_numpy(_lib.time_basis([7.0])).to(dev)
    opts, _keep = _opts(mode, full, basis)
    for i, x in enumerate((0.25, np.nextafter(np.float32(0.25), np.float32(0)), np.nextafter(np.float32(0.5), np.float32(1)))):
        fwd = [0.0, 0.0, 0.0]
        eye = [float(x)] * 3
        eye[i], fwd[i] = -0.8, 1.0
        fwd[(i + 1) % 3] = 3e-8
        cam = synth.Camera(eye=tuple(eye), fwd=tuple(fwd), up=tuple(float(a == (i + 2) % 3) for a in range(3)),
                           fov_y_deg=25.0, width=w, height=h, time=7.0)
        note(f"camera along axis {i} {mode} {w}x{h}")
        _, T = _lib.render(full, [cam], opts, want_T=True, decode=False)
        torch.cuda.synchronize()
        o, d = oracle.camera_rays(cam)
        err = np.abs(T.cpu().numpy().reshape(-1).astype(np.float64) -
                     np.exp(-SIGMA * _chord(np.asarray(o), np.asarray(d))))
        # the oracle's directions are FP64: a chord that leaves through another face moves continuously
        assert err.max() <= 5e-5, (i, int((err > 5e-5).sum()), err.max())
