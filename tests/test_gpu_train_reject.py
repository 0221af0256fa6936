"""A training step whose batch is rejected on the device leaves loss and gradient as they were."""
import ctypes

import numpy as np
import pytest

from paper_1903_10741_amd import workloads as W
from test_gpu_surrogate import _ffs, _params, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", ["gene", "target"])
def test_rejected_batch_writes_no_loss_or_grad(bad):
    torch, ffsga = _ffs()
    _say("rejected batch:", bad)
    n, B = 9, 70
    th, _ = _params(n)
    m = ffsga.Surrogate(th)
    inst = W.random_instance(n, n_jobs=n, n_stages=3, machines=2, p_max=30)
    feats = m.features(ffsga.DeviceInstance.from_host(inst))
    prio = torch.from_numpy(W.random_population(n, B, n)).cuda()
    tgt = torch.from_numpy(np.random.default_rng(n).normal(size=B).astype(np.float32)).cuda()
    if bad == "gene":
        prio[3, 4] = 0
    else:
        tgt[69] = float("nan")
    loss = torch.full((1,), 5.0, device="cuda")
    grad = torch.full((ffsga.SG_PARAMS,), 7.0, device="cuda")
    ws = torch.zeros(ffsga._lib.sg_train_workspace_size(n, B), dtype=torch.uint8, device="cuda")
    before = m.theta.clone()
    ptr = [ctypes.c_void_p(t.data_ptr()) for t in (feats, prio, tgt, loss, grad, ws)]
    assert ffsga._lib.sg_train_step(ctypes.byref(m.s), ptr[0], n, ptr[1], ptr[2], B, 1e-3, ptr[3], ptr[4],
                                    ptr[5], ws.numel(), ffsga._stream()) == 0
    torch.cuda.synchronize()
    assert float(loss) == 5.0 and bool((grad == 7.0).all()) and torch.equal(m.theta, before)
