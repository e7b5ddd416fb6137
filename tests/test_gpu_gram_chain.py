"""The one-workgroup chain of the moment form at the edges of its thread layouts (4 threads per row up to 64 features, 8 beyond;
16- and 4-byte parts of a row with every remainder), for every update rule, over launches of more steps than one block of
Adam's bias corrections holds.  fp32 sums of at most p products per step, as in the other tests of this form: 1e-4."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("p", [1, 3, 15, 16, 17, 33, 47, 63, 64, 65, 128])
def test_layouts_and_rules(p, kind):
    import torch
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = wl.CONFIGS["cfg2"].scaled(name="case", N=2010, p=p, N0=1005, n=25, T=5, R=1, x_cov="identity")   # 164 steps, then 41
    X, y = wl.dataset(w)
    rate = 0.01 if kind == 3 else 0.1 / (p + 10)
    opts = dict(momentum=0.8, beta1=0.9, beta2=0.99, eps=1e-6)
    ref = O.BMGD(w.model, p, w.n, rate, w.T)
    if kind:
        ref.set_optimizer(kind, **opts)
    table = np.linspace(rate, rate / 5, 300).astype(np.float32) if p % 2 else None
    ctx = B.Context(p, w.N0, w.n, rate, w.T, model=w.model, chain=B.BMGD_CHAIN_GRAM, optimizer=kind, **opts)
    if table is not None:
        ref.set_lr_schedule(table)
        ctx.set_lr_schedule(table)
    xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    s = torch.cuda.Stream()
    for k in range(2):
        lo, hi = k * w.N0, (k + 1) * w.N0
        ref.run_buffer(X[lo:hi], y[lo:hi])
        ctx.run_device_buffer(xd[lo:hi].clone(), yd[lo:hi].clone(), w.N0, s)
        ctx.sync()
    got, st = ctx.get_theta(), ctx.stats()
    ctx.close()
    assert st.steps == 2 * 5 * 41
    assert rel_l2(got, ref.theta) <= 1e-4
