"""bmgd_eval_loss against the fp64 oracle's loss, for the three models, and its use along a run: the global loss
of a mini-batch run with a small learning rate goes down from iteration to iteration."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import rel_l2

pytestmark = pytest.mark.gpu


def _ctx_with_theta(w, theta):
    import paper_2312_08728_amd as B
    ctx = B.Context(w.p, w.N0, w.n, w.alpha, w.T, model=w.model, n_classes=w.C)
    ctx.set_theta(theta)
    return ctx


@pytest.mark.parametrize("model,p,rows", [(wl.LINEAR, 10, 1), (wl.LINEAR, 100, 5000), (wl.LOGISTIC, 200, 7777),
                                          (wl.LOGISTIC, 4096, 300), (wl.LINEAR, 37, 70_001)])
def test_glm_loss_matches_oracle(model, p, rows):
    import torch
    from oracle import bmgd as O
    base = wl.CONFIGS["cfg3" if model == wl.LOGISTIC else "cfg2"]
    w = base.scaled(name="case", model=model, N=rows, p=p, N0=max(rows, 2), n=max(min(rows, 100), 1), T=1, R=1, x_cov="identity")
    X, y = wl.dataset(w)
    theta = (np.random.default_rng(1).standard_normal(p) / np.sqrt(p)).astype(np.float32)
    want = O.loss(model, X.astype(np.float64), y.astype(np.float64), theta.astype(np.float64))
    ctx = _ctx_with_theta(w, theta)
    got = ctx.eval_loss(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), rows)
    ctx.close()
    assert abs(got - want) <= 2e-5 * abs(want)


def test_softmax_loss_matches_oracle():
    import torch
    from oracle import bmgd as O
    w = wl.CONFIGS["cfg5"].scaled(name="case", N=3000, p=200, C=130, N0=1500, n=256, T=1, R=1)
    X, y = wl.dataset(w)
    W = (np.random.default_rng(2).standard_normal((w.p, w.C)) * 0.05).astype(np.float32)
    want = O.loss(w.model, O.to_f64(X), y, W.astype(np.float64))
    ctx = _ctx_with_theta(w, W)
    got = ctx.eval_loss(torch.from_numpy(X.view(np.int16)).cuda(), torch.from_numpy(y).cuda(), 3000)
    ctx.close()
    assert abs(got - want) <= 2e-3 * abs(want)                 # logits from the bf16 copy of W


def test_global_loss_goes_down_over_iterations():
    import torch
    import paper_2312_08728_amd as B
    w = wl.CONFIGS["cfg3"].scaled(name="case", N=40_000, p=50, N0=10_000, n=500, T=2, R=4, alpha=0.05)
    X, y = wl.dataset(w)
    xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    ctx = B.Context(w.p, w.N0, w.n, w.alpha, w.T, model=w.model)
    s = torch.cuda.Stream()
    losses = [ctx.eval_loss(xd, yd, w.N)]
    for r in range(w.R):
        for k in range(4):
            ctx.run_device_buffer(xd[k * w.N0:(k + 1) * w.N0], yd[k * w.N0:(k + 1) * w.N0], w.N0, s)
        losses.append(ctx.eval_loss(xd, yd, w.N, s))
    ctx.close()
    assert abs(losses[0] - np.log(2.0)) < 1e-6                  # theta = 0: every row costs log 2
    assert all(b < a for a, b in zip(losses, losses[1:])), losses


@pytest.mark.parametrize("p", [1, 2, 3, 6, 36, 129, 258, 1000, 1023, 2046, 4095])
def test_loss_at_every_row_layout_and_remainder(p):
    """Each vector width and number of chunks per lane (and rows beyond them), with rows that fill no wavefront, one
    group exactly, and one more: sums of p products in fp32 (2^-24 sqrt(p) relative to the terms, far below 2e-5)."""
    import torch
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    rng = np.random.default_rng(p)
    theta = (rng.standard_normal(p) / np.sqrt(p)).astype(np.float32)
    for model, rows in ((wl.LINEAR, 1), (wl.LOGISTIC, 31), (wl.LOGISTIC, 2048), (wl.LINEAR, 2049)):
        X = rng.standard_normal((rows, p)).astype(np.float32)
        y = (rng.random(rows) < 0.5).astype(np.float32)
        rc = B.bmgd_eval_loss_static(model, torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(),
                                     torch.from_numpy(theta).cuda(), rows, p, None, out)
        assert rc == B.BMGD_OK
        want = O.loss(model, X.astype(np.float64), y.astype(np.float64), theta.astype(np.float64))
        assert abs(float(out.cpu()[0]) - want) <= 2e-5 * abs(want), (p, model, rows)


@pytest.mark.parametrize("p,C,batch,rows", [
    (8, 2, 64, 1),                 # one row
    (200, 130, 64, 1024),          # exactly what the scratch of 64-row mini-batches holds
    (200, 130, 64, 1025),          # one row in a second launch
    (72, 300, 100, 3100),          # several launches, the last one ragged
    (2048, 40, 300, 500),          # few tiles: K split over workgroups
    (520, 1100, 128, 700),         # more than 1,024 classes, K not a multiple of the tile
])
def test_softmax_loss_in_one_or_several_launches(p, C, batch, rows):
    """Logits from the bf16 copy of W, taken from the same copy by the reference: what is left are sums of p products in fp32
    (2^-24 sqrt(p) of their size) and a logarithm, far below 1e-5."""
    import torch
    import paper_2312_08728_amd as B
    gen = torch.Generator().manual_seed(p + rows)
    X = torch.randn((rows, p), generator=gen).bfloat16()
    y = torch.randint(0, C, (rows,), generator=gen, dtype=torch.int32)
    W = (torch.randn((p, C), generator=gen) / p ** 0.5).bfloat16()
    want = torch.nn.functional.cross_entropy(X.double() @ W.double(), y.long()).item()
    ctx = B.Context(p, max(rows, batch), batch, 0.1, 1, model=B.BMGD_SOFTMAX, n_classes=C)
    ctx.set_theta(W.float().numpy())
    got = ctx.eval_loss(X.cuda(), y.cuda(), rows)
    ctx.close()
    assert abs(got - want) <= 1e-5 * abs(want)


@pytest.mark.parametrize("bad", [np.inf, -np.inf])
@pytest.mark.parametrize("p", [3, 6, 37, 100, 130, 516, 1000, 2046])
def test_an_infinite_predictor_gives_an_infinite_loss(p, bad):
    """Least squares: (x'theta - y)^2 / 2 with one infinite product is infinite, at row lengths that do not fill the lanes which
    hold a row (what those hold beyond p takes no part, whatever the row's first column is)."""
    import torch
    import paper_2312_08728_amd as B
    rng = np.random.default_rng(p)
    X = rng.standard_normal((50, p)).astype(np.float32)
    X[7, 0] = bad
    y = rng.standard_normal(50).astype(np.float32)
    theta = (rng.standard_normal(p) / np.sqrt(p)).astype(np.float32)
    xd, yd, out = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), torch.empty(1, dtype=torch.float64, device="cuda")
    assert B.bmgd_eval_loss_static(B.BMGD_LINEAR, xd, yd, torch.from_numpy(theta).cuda(), 50, p, None, out) == B.BMGD_OK
    assert float(out.cpu()[0]) == np.inf
    ctx = B.Context(p, 50, 10, 0.1, 1)
    ctx.set_theta(theta)
    got = ctx.eval_loss(xd, yd, 50)
    ctx.close()
    assert got == np.inf
