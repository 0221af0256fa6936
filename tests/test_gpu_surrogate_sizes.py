"""A training step at the sizes where its tiles (64 table rows, 256 per dW2 partial), chunks (64
and 256 chromosomes) and check blocks (4096 genes) end, against the float64 oracle within its
forward and gradient bounds; a gene or target that the check must find in the last place."""
import numpy as np
import pytest

from oracle import surrogate as S
from paper_1903_10741_amd import workloads as W
from test_gpu_surrogate import _ffs, _params, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,B", [(1, 1), (7, 64), (8, 65), (16, 255), (17, 257), (65, 63), (70, 130)])
def test_train_step_sizes(n, B):
    torch, ffsga = _ffs()
    _say("train step n", n, "batch", B)
    inst = W.random_instance(n, n_jobs=n, n_stages=3, machines=2, p_max=30)
    th, p = _params(n)
    m = ffsga.Surrogate(th)
    feats = m.features(ffsga.DeviceInstance.from_host(inst))
    prio = W.random_population(n, B, n)
    tgt = np.random.default_rng(n).normal(size=B).astype(np.float32)
    loss, grad = m.train_step(feats, torch.from_numpy(prio), torch.from_numpy(tgt), 1e-3,
                              want_grad=True)
    L, g, f = S.loss_and_grad(p, S.job_features(inst), prio, tgt.astype(np.float64))
    bnd = S.grad_bound(p, f)
    got = S.unflatten(grad.cpu().numpy())
    for k in g:
        err = np.abs(got[k].astype(np.float64).reshape(g[k].shape) - g[k])
        assert (err <= bnd[k] + 1e-30).all(), (k, float((err - bnd[k]).max()))
    e_d = S.forward_bound(p, f, "pool") + S.U32 * np.abs(f["target"])
    dd = np.abs(f["y"] - f["target"])
    e_L = np.mean(2 * dd * e_d + e_d ** 2) + (S._gamma(B) + 2 * S.U32) * np.mean((dd + e_d) ** 2)
    assert abs(float(loss.item()) - L) <= e_L
    # the last gene, then the last target, made invalid: no parameter changes
    before = m.theta.clone()
    for bad in ("gene", "target"):
        bp, bt = prio.copy(), tgt.copy()
        if bad == "gene":
            bp[-1, -1] = n + 1
        else:
            bt[-1] = np.inf
        m.train_step(feats, torch.from_numpy(bp), torch.from_numpy(bt), 1e-3)
        assert torch.equal(m.theta, before)
