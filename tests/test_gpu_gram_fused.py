"""The moment form in one kernel (few features, few and small mini-batches, the mode left to the library): partitions, matrices and
chain of a launch.  fp32 sums of at most n products per entry and p per update, as in the other tests of this form: 1e-4."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import rel_l2

pytestmark = pytest.mark.gpu


def _run(p, N0, n, T, kind, table=None, subset=None, **kw):
    import torch
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = wl.CONFIGS["cfg2"].scaled(name="case", N=2 * N0, p=p, N0=N0, n=n, T=T, R=1, x_cov="identity")
    X, y = wl.dataset(w)
    rate = 0.01 if kind == 3 else 0.1 / (p + 10)
    opts = dict(momentum=0.8, beta1=0.9, beta2=0.99, eps=1e-6)
    ref = O.BMGD(w.model, p, w.n, rate, w.T)
    ctx = B.Context(p, w.N0, w.n, rate, w.T, model=w.model, optimizer=kind, **opts, **kw)
    if kind:
        ref.set_optimizer(kind, **opts)
    if table is not None:
        sched = np.linspace(rate, rate / 5, table).astype(np.float32)
        ref.set_lr_schedule(sched)
        ctx.set_lr_schedule(sched)
    xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    idx = None if subset is None else torch.from_numpy(subset).cuda()
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    keep = []
    for k in range(2):
        lo, hi = k * w.N0, (k + 1) * w.N0
        xk, yk = xd[lo:hi].clone(), yd[lo:hi].clone()
        torch.cuda.synchronize()
        keep.append((xk, yk))
        if subset is not None:
            ctx.set_row_subset(idx, len(subset))
            ref.run_buffer(X[lo:hi][subset], y[lo:hi][subset])
        else:
            ref.run_buffer(X[lo:hi], y[lo:hi])
        ctx.run_device_buffer(xk, yk, w.N0, s)
    got, st = ctx.get_theta(), ctx.stats()
    ctx.close()
    return got, ref.theta, st


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("p", [1, 3, 4, 15, 16, 17, 31, 32, 33, 47, 48, 62, 63])
def test_layouts_and_rules(p, kind):
    """Every tile and chain layout; seven mini-batches, the last one of 6 rows, in launches of 28 and 7 steps."""
    got, want, st = _run(p, N0=6 * 131 + 6, n=131, T=5, kind=kind, table=50 if p % 2 else None)
    assert st.prep_launches == 0 and st.chain_launches == 4 and st.n_workgroups == 1 and st.steps == 2 * 5 * 7
    assert rel_l2(got, want) <= 1e-4


@pytest.mark.parametrize("N0,n,T,kind", [(126, 2, 4, 0),      # one-row shares, most steps a wavefront's rows are few for
                                         (504, 2, 4, 1),      # 1,008 steps in a launch: the most (with state)
                                         (512, 512, 1, 0),    # one mini-batch of the largest size: 64 rows a wavefront
                                         (1030, 511, 3, 0),   # 64 and 63 rows a wavefront; a last mini-batch of 8 rows
                                         (521, 260, 2, 0)])   # 36 rows: a second request of four rows; a last mini-batch of one row
def test_shapes(N0, n, T, kind):
    got, want, st = _run(1, N0=N0, n=n, T=T, kind=kind)
    assert st.prep_launches == 0 and rel_l2(got, want) <= 1e-4


@pytest.mark.parametrize("p,most", [(1, 256), (32, 256), (33, 160), (48, 160), (49, 128), (63, 128)])
def test_plain_steps_up_to_where_products_are_faster(p, most):
    """At the line and one mini-batch beyond it, by mini-batches and by passes."""
    n = 2 * p
    for M, T in ((most // 4, 4), (most // 4 + 1, 4), (most // 2, 2), (most // 2 + 1, 2)):
        got, want, st = _run(p, N0=M * n, n=n, T=T, kind=0)
        assert (st.prep_launches == 0) == (M * T <= most) and rel_l2(got, want) <= 1e-4


def test_more_passes_than_the_context_was_made_with():
    """The form is chosen for the passes of the context; a run of more of them fits its workspace (1,000 steps in a launch)."""
    import torch
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    p, n, N0 = 3, 8, 2000
    w = wl.CONFIGS["cfg2"].scaled(name="case", N=N0, p=p, N0=N0, n=n, T=1, R=1, x_cov="identity")
    X, y = wl.dataset(w)
    ctx, ref = B.Context(p, N0, n, 0.01, 1, model=w.model), O.BMGD(w.model, p, n, 0.01, 1)
    xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    torch.cuda.synchronize()
    for T in (1, 4, 5):
        ctx.set_passes(T)
        ref.T = T
        ctx.run_device_buffer(xd, yd, N0)
        ref.run_buffer(X, y)
    got, st = ctx.get_theta(), ctx.stats()
    ctx.close()
    assert st.prep_launches == 0 and st.chain_launches == 4 and rel_l2(got, ref.theta) <= 1e-4


def test_beyond_the_rule_other_kernels_run():
    for N0, n in ((506, 2), (1030, 513)):                # 1,012 steps in a launch of four passes; a mini-batch of 513 rows
        got, want, st = _run(1, N0=N0, n=n, T=4, kind=0)
        assert st.prep_launches > 0 and rel_l2(got, want) <= 1e-4


def test_row_subset():
    rng = np.random.default_rng(3)
    got, want, st = _run(20, N0=900, n=100, T=3, kind=0, subset=rng.choice(900, 333, replace=False).astype(np.int32))
    assert st.prep_launches == 0 and rel_l2(got, want) <= 1e-4


# Calls that name a stream, in the order of their enqueueing: run over a resident buffer (r), over a loaded one (l), the same with
# its passes left to the library (a), theta folded into the running average (s); "zX" keeps stream X busy for a while first, so that without an order of its own what follows on
# the other stream would overtake what waits behind it.
ORDERS = {
    "resident": ["zA"] + ["rA", "rB"] * 15 + ["zB", "rB", "rA"],
    "adaptive_behind_run": ["zA", "lA", "aB", "zB", "lB", "aA"],
    "run_behind_adaptive": ["zB", "aB", "lA", "rB", "zA", "aA", "rB"],
    "run_behind_average": ["rA", "rB", "zB", "sB", "rA", "zA", "sA", "rB", "sB", "aA"],
    "average_behind_run_elsewhere": ["rA", "zB", "rB", "sA", "rA", "zA", "aA", "sB", "sA"],
}


@pytest.mark.parametrize("order", sorted(ORDERS))
@pytest.mark.parametrize("kind", [0, 1])
def test_calls_on_two_streams_follow_one_another(kind, order):
    """Nothing is waited for on the host until the end; theta after every sequence, and the statistics' count of launches."""
    import torch
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    p, N0, n, T = 12, 2000, 100, 2
    w = wl.CONFIGS["cfg2"].scaled(name="case", N=4 * N0, p=p, N0=N0, n=n, T=T, R=1, x_cov="identity")
    X, y = wl.dataset(w)
    rate = 0.1 / (p + 10)
    ctx = B.Context(p, N0, n, rate, T, model=w.model, optimizer=kind, momentum=0.8)
    parts = [slice(k * N0, (k + 1) * N0) for k in range(4)]
    xp, yp = torch.from_numpy(X).pin_memory(), torch.from_numpy(y).pin_memory()
    dev = [(xp[part].cuda(), yp[part].cuda()) for part in parts]
    ss = {"A": torch.cuda.Stream(), "B": torch.cuda.Stream()}
    copy = torch.cuda.Stream()
    torch.cuda.synchronize()
    calls = [c for c in ORDERS[order] if c[0] != "z"]
    k = 0
    for what, which in ORDERS[order]:
        if what == "z":
            with torch.cuda.stream(ss[which]):
                torch.cuda._sleep(2_000_000)
            continue
        if what == "s":
            ctx.swa_update(ss[which])
            continue
        part = parts[k % 4]
        k += 1
        if what == "r":
            ctx.run_device_buffer(*dev[(k - 1) % 4], N0, ss[which])
            continue
        ctx.load_buffer_async(xp[part], yp[part], N0, copy)
        if what == "l":
            ctx.run_buffer(ss[which])
        else:
            assert ctx.run_buffer_adaptive(ss[which], None, None, 0, None, T, T) == T
    averages = sum(c[0] == "s" for c in calls)
    if averages:                                         # (fetched first: nothing has been waited for yet)
        avg, count = ctx.get_swa()
    got, st = ctx.get_theta(), ctx.stats()
    ctx.close()
    ref = O.BMGD(w.model, p, n, rate, T)
    if kind:
        ref.set_optimizer(kind, momentum=0.8)
    k = 0
    for what, _ in calls:
        if what == "s":
            ref.swa_update()
            continue
        ref.run_buffer(X[parts[k % 4]], y[parts[k % 4]])
        k += 1
    if averages:
        assert count == averages and rel_l2(avg, ref.swa) <= 1e-4
    # (an adaptive run is one launch a pass)
    assert st.prep_launches == 0 and st.chain_launches == sum({"a": T, "s": 0}.get(c[0], 1) for c in calls)
    assert rel_l2(got, ref.theta) <= 1e-4
