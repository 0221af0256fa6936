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


@pytest.mark.parametrize("n", [1, 63, 64, 65, 256])
def test_scores_of_a_large_count_keep_their_bits(n):
    """32767 chromosomes are scored one a wave, 32768 and more in blocks of 128 with the table in
    LDS: each gets the same bits from both, invalid genes a NaN, and no score is written past the
    count."""
    torch, ffsga = _ffs()
    _say("scores of a large count, n", n)
    th, _ = _params(n)
    m = ffsga.Surrogate(th)
    inst = W.random_instance(n, n_jobs=n, n_stages=2, machines=2, p_max=9)
    table = m.score_table(m.features(ffsga.DeviceInstance.from_host(inst)), n)
    count = 32768 + 131
    prio = torch.from_numpy(W.random_population(n, count, n)).cuda()
    prio[[5, 130, count - 1], [0, n // 2, n - 1]] = torch.tensor([0, n + 1, -7], dtype=torch.int32).cuda()
    want = torch.cat([m.score(table, prio[:20000]), m.score(table, prio[20000:])])
    got = m.score(table, prio)
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    assert torch.isnan(got).sum() == 3


@pytest.mark.parametrize("count,group", [(1, 1), (300, 255), (513, 257), (4096, 4096), (8193, 4096),
                                         (4097, 4097), (9000, 9000)])
def test_targets_sizes(count, group):
    """Groups on either side of the 256 runs and of the 4096 entries whose logarithms are kept."""
    torch, ffsga = _ffs()
    _say("targets of", count, "in groups of", group)
    obj = np.random.default_rng(count).integers(1, 10**6, size=count).astype(np.int64)
    got = ffsga.Surrogate(W.surrogate_init(0)).targets(torch.from_numpy(obj), group)
    want = S.targets(obj, group)
    assert (np.abs(got.cpu().numpy().astype(np.float64) - want) <= S.U32 * np.abs(want) + 1e-9).all()
