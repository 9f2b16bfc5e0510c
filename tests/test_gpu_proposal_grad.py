"""The proposal network's batch gradient at the sizes where its blocking can go
wrong: single rays, around one 64-ray chunk, and past 256 chunks (a block's
second turn), against the FP64 oracle at the bounds of the 3000-ray test."""
import numpy as np
import pytest

from oracle import mlp
from paper_2202_08614_amd import _lib, synth
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 16384, 16384 + 64 + 3])
def test_batch_gradient_edges(n):
    import torch
    dev = require_gpu()
    rng = np.random.default_rng(n)
    p = np.concatenate([np.asarray(synth.mlp_init(3), np.float32).ravel()[:mlp.N_PARAMS], np.zeros(1, np.float32)])
    w = mlp.from_flat(p[:mlp.N_PARAMS].astype(np.float64))
    X = rng.uniform(-1.0, 1.0, (4000, 7)).astype(np.float32)
    hit = (rng.random((4000, 1)) < 0.5).astype(np.float32)
    Y = np.concatenate([hit, np.sort(rng.random((4000, 2)).astype(np.float32), 1) * hit], 1).astype(np.float32)
    o, (_, z1, _, z2, _) = mlp.forward(w, X.astype(np.float64))
    u = np.abs(Y[:, 1:] - mlp.sigmoid(o[:, 1:]))
    ok = (np.abs(z1).min(1) > 1e-3) & (np.abs(z2).min(1) > 1e-3) & ((Y[:, 0] < 0.5) | (u.min(1) > 1e-3))
    idx = rng.choice(np.nonzero(ok)[0], n).astype(np.int32)
    Pd, Xd, Yd = (torch.from_numpy(a).to(dev) for a in (p, X, Y))
    grad = torch.zeros_like(Pd)
    loss = torch.zeros(1, dtype=torch.float32, device=dev)
    size = _lib.mlp_workspace(n, dev).numel()
    ws = torch.full((size + 64,), float("nan"), device=dev)
    note(f"fpo_mlp_loss_grad n={n}")
    _lib.mlp_loss_grad(Pd, Xd, Yd, grad, loss, ws, idx=torch.from_numpy(idx).to(dev))
    torch.cuda.synchronize()
    assert bool(torch.isnan(ws[size:]).all())
    rows, cnt = np.unique(idx, return_counts=True)
    xb, yb = X[rows].astype(np.float64), Y[rows].astype(np.float64)
    ob, cb = mlp.forward(w, xb)
    per = np.array([mlp.loss_and_grad_out(ob[i:i + 1], yb[i:i + 1])[0] for i in range(len(rows))])
    want_loss = float((per * cnt).sum() / n)
    g_out = np.concatenate([mlp.loss_and_grad_out(ob[i:i + 1], yb[i:i + 1])[1] for i in range(len(rows))])
    g_out = g_out * (cnt / n)[:, None]
    want = mlp.to_flat(mlp.backward(w, cb, g_out))
    gb, _, a1b, _, a2b = cb
    d2 = np.abs(g_out) @ np.abs(w["W3"]).T
    d1 = d2 @ np.abs(w["W2"]).T
    ones = np.ones((len(rows), 1))
    mag = np.concatenate([(np.hstack([np.abs(gb), ones]).T @ d1).ravel(),
                          (np.hstack([a1b, ones]).T @ d2).ravel(),
                          (np.hstack([a2b, ones]).T @ np.abs(g_out)).ravel()])
    got = grad.cpu().numpy()
    assert np.all(np.abs(got[:mlp.N_PARAMS] - want) <= 2.0 ** -14 * mag + 1e-12)
    assert got[mlp.N_PARAMS] == 0.0
    assert abs(float(loss.item()) - want_loss) <= 1e-5 * want_loss
    # parameters that are not 16-byte aligned: the same sums
    shifted = torch.cat([torch.zeros(1, device=dev), Pd])[1:]
    assert shifted.data_ptr() % 16 != 0
    again = torch.zeros_like(grad)
    _lib.mlp_loss_grad(shifted, Xd, Yd, again, loss, ws, idx=torch.from_numpy(idx).to(dev))
    torch.cuda.synchronize()
    assert torch.equal(again, grad)
