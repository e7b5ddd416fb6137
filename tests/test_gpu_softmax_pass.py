"""The persistent softmax kernel of large mini-batches (logits, residual and update of many steps in one launch) at the edges of
its tiles, against the fp64 oracle within the bound of the bf16 path (2e-3: bf16 copy of W, bf16 residual; 5e-3 with Adam, which
normalises their rounding), and against the three launches, whose roundings are the same up to the order of fp32 sums."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import gpu_run, oracle_run, rel_l2

pytestmark = pytest.mark.gpu


def _case(N, p, C, N0, n, T=2, R=1, alpha=0.05):
    return wl.CONFIGS["cfg5"].scaled(name="case", N=N, p=p, C=C, N0=N0, n=n, T=T, R=R, alpha=alpha)


@pytest.mark.parametrize("N,p,C,N0,n", [
    (300, 1032, 10, 200, 64),          # one tile of classes and rows; features 8 beyond an operand tile
    (310, 1064, 129, 200, 65),         # one class in the second tile, one row beyond an operand tile; a last mini-batch of 5 rows
    (1300, 1096, 130, 1250, 600),      # a last mini-batch of 50 rows: four of five row tiles are empty in it; a shorter buffer
    (4200, 200, 40, 4200, 1100),       # many rows of few features: the logits' depth is hardly split
    (4100, 136, 300, 4100, 2048),      # most rows
    (700, 2304, 260, 650, 129),        # three tiles of classes, eight parts of the depth
    (900, 2048, 1000, 900, 300),       # 64 features a tile
    (2100, 3072, 1000, 2100, 1024),    # 96 features a tile, every workgroup one item of each phase
    (500, 4096, 1000, 500, 250),       # 128 features a tile
    (400, 4104, 2000, 400, 200),       # several rounds of tiles
])
def test_edges(N, p, C, N0, n):
    import paper_2312_08728_amd as B
    w = _case(N, p, C, N0, n)
    X, y = wl.dataset(w)
    want = oracle_run(w, X, y)
    got, st = gpu_run(w, X, y)
    assert st.steps == w.steps and np.isfinite(got).all()
    assert rel_l2(got, want) <= 2e-3
    three, _ = gpu_run(w, X, y, chain=B.BMGD_CHAIN_LAUNCH)
    assert rel_l2(got, three) <= 2e-3


@pytest.mark.parametrize("p,n", [(p, 1100) for p in (40, 72, 136, 200, 264, 328, 392, 456)] + [(1064, n) for n in (50, 100, 150, 200, 300, 350, 400, 500)])
def test_one_operand_tile_to_eight(p, n):
    """The depth of the logits, and of the update, in every number of operand tiles that its pipeline starts or ends differently with."""
    w = _case(n + 30, p, 130, n + 30, n)
    X, y = wl.dataset(w)
    got, st = gpu_run(w, X, y)
    assert st.steps == w.steps and rel_l2(got, oracle_run(w, X, y)) <= 2e-3


@pytest.mark.parametrize("N,p,C,N0,n,optimizer", [
    (310, 1064, 129, 200, 65, 0),
    (310, 1064, 129, 200, 65, 1),
    (900, 1296, 300, 700, 200, 2),
    (900, 2048, 1000, 700, 300, 3),
    (500, 3072, 1000, 400, 200, 3),    # 96 features a tile
    (500, 4096, 1000, 400, 200, 3),    # 128
    (500, 4096, 1000, 400, 200, 1),
])
def test_update_rules_and_one_workgroup_alone(N, p, C, N0, n, optimizer):
    """A table of rates, two buffers of different size and a run behind them, five passes (two launches a run), against the launches; and
    by one workgroup alone (a limit on waits that leaves no time to meet): the same sums in the same order, the same bits."""
    import torch
    import paper_2312_08728_amd as B
    w = _case(N, p, C, N0, n, T=5)
    X, y = wl.dataset(w)
    xd, yd = torch.from_numpy(X.view(np.int16)).cuda(), torch.from_numpy(y).cuda()
    s = torch.cuda.Stream()
    top = 0.002 if optimizer == 3 else 0.02
    got = []
    for chain, limit in ((B.BMGD_CHAIN_AUTO, 0), (B.BMGD_CHAIN_AUTO, 1), (B.BMGD_CHAIN_LAUNCH, 0)):
        ctx = B.Context(w.p, w.N0, w.n, top, w.T, model=w.model, n_classes=w.C, chain=chain, optimizer=optimizer, barrier_timeout_us=limit)
        ctx.set_lr_schedule(np.linspace(top, top / 10, 9).astype(np.float32))
        for k in (0, 1, 0):
            lo, hi = wl.buffer_rows(w, k)
            ctx.run_device_buffer(xd[lo:hi], yd[lo:hi], hi - lo, s)
        got.append((ctx.get_theta(), ctx.eval_loss(xd, yd, w.N, s)))      # (the loss reads the bf16 copy the kernel leaves)
        ctx.close()
    assert np.isfinite(got[0][0]).all() and got[0][0].any()
    assert np.array_equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]
    # Adam: see test_gpu_softmax_chain.py (the sign of a gradient near zero decides its first update)
    assert rel_l2(got[0][0], got[2][0]) <= (1.2e-2 if optimizer == 3 else 2e-3)
    assert abs(got[0][1] - got[2][1]) <= 2e-3 * abs(got[2][1])


def test_contexts_that_compete_for_the_compute_units():
    """Two softmax runs and a long run of the persistent logistic kernel on streams of their own: whichever workgroups find room, every
    run ends as it does with the device to itself."""
    import torch
    import paper_2312_08728_amd as B
    w = _case(4000, 1536, 700, 4000, 500)
    X, y = wl.dataset(w)
    xd, yd = torch.from_numpy(X.view(np.int16)).cuda(), torch.from_numpy(y).cuda()
    v = wl.CONFIGS["cfg3"].scaled(name="other", N=200_000, p=200, N0=200_000, n=4096, T=4, R=1)
    VX, vy = wl.dataset(v)
    vx, vyd = torch.from_numpy(VX).cuda(), torch.from_numpy(vy).cuda()
    streams = [torch.cuda.Stream() for _ in range(3)]
    results = []
    for together in (False, True):
        soft = [B.Context(w.p, w.N0, w.n, w.alpha, w.T, model=w.model, n_classes=w.C, seed=i) for i in range(2)]
        glm = B.Context(v.p, v.N0, v.n, v.alpha, v.T, model=v.model, chain=B.BMGD_CHAIN_PERSISTENT)
        torch.cuda.synchronize()
        for _ in range(3):
            for ctx, s in [(glm, streams[2])] + list(zip(soft, streams)):
                ctx.run_device_buffer(*((vx, vyd, v.N0) if ctx is glm else (xd, yd, w.N0)), s)
                if not together:
                    ctx.sync()
        results.append([c.get_theta() for c in soft + [glm]])
        for c in soft + [glm]:
            c.close()
    for a, b in zip(*results):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_values_that_are_not_finite(bad):
    """They spread as in the launches, and classes that fill up the last tile stay zero: after bmgd_set_theta a run over clean rows is that
    of a new context."""
    import torch
    import paper_2312_08728_amd as B
    w = _case(260, 1048, 130, 260, 130, T=1)
    X, y = wl.dataset(w)
    clean = torch.from_numpy(X.view(np.int16)).view(torch.bfloat16).cuda()
    x = clean.clone()
    x[5, 3] = float(bad)
    yd, s = torch.from_numpy(y).cuda(), torch.cuda.Stream()
    w0 = (np.random.default_rng(0).standard_normal((w.p, w.C)) * 0.05).astype(np.float32)
    runs = []
    for chain in (B.BMGD_CHAIN_AUTO, B.BMGD_CHAIN_LAUNCH):
        ctx = B.Context(w.p, 260, 130, 0.05, 1, model=w.model, n_classes=w.C, chain=chain)
        ctx.set_theta(w0)
        ctx.run_device_buffer(x, yd, 260, s)
        runs.append(ctx.get_theta())
        if chain == B.BMGD_CHAIN_AUTO:
            ctx.set_position(0)
            ctx.set_theta(w0)
            ctx.run_device_buffer(clean, yd, 260, s)
            again = ctx.get_theta()
        ctx.close()
    assert np.isnan(runs[0]).any() and np.array_equal(np.isnan(runs[0]), np.isnan(runs[1]))
    ctx = B.Context(w.p, 260, 130, 0.05, 1, model=w.model, n_classes=w.C)
    ctx.set_theta(w0)
    ctx.run_device_buffer(clean, yd, 260, s)
    assert np.array_equal(again, ctx.get_theta()) and np.isfinite(again).all()
    ctx.close()


def _streams(k):
    """Streams whose work runs side by side (HIP spreads streams over a few hardware queues)."""
    import time
    import torch
    got = []
    for _ in range(10):
        s, free = torch.cuda.Stream(), True
        for other in got:
            torch.cuda.synchronize()
            with torch.cuda.stream(other):
                torch.cuda._sleep(40_000_000)
            e = torch.cuda.Event()
            e.record(s)
            time.sleep(0.003)
            free = free and e.query()
        torch.cuda.synchronize()
        if free:
            got.append(s)
        if len(got) == k:
            return got
    pytest.fail("no streams that run side by side")


class _Holder:
    """A run of the logistic persistent kernel that keeps `units` compute units for about `ms` milliseconds in one launch: 3.1 us an update
    on 152 to 256 of them."""

    def __init__(self, units, ms):
        import torch
        import paper_2312_08728_amd as B
        self.rows = 64 * int(ms / 4 / 3.13e-3)
        self.x, self.y = torch.randn((self.rows, 16), device="cuda"), torch.ones(self.rows, device="cuda")
        self.ctx = B.Context(16, self.rows, 64, 0.01, 4, model=B.BMGD_LOGISTIC, chain=B.BMGD_CHAIN_PERSISTENT, n_workgroups=units)
        assert self.ctx.stats().n_workgroups == units
        self.free = torch.cuda.Event(enable_timing=True)

    def start(self, stream):
        import time
        self.ctx.run_device_buffer(self.x, self.y, self.rows, stream)
        self.free.record(stream)
        time.sleep(0.004)
        assert not self.free.query()


def test_a_persistent_kernel_gets_the_units_that_it_waits_for():
    """Softmax runs on the eight compute units that another context leaves it, then the next run of that stream wants all of them, with a limit
    of 50 ms: the softmax run (100 updates a pass, 0.7 ms each on eight units) lets go of them in time."""
    import torch
    import paper_2312_08728_amd as B
    p, C, n, M = 2048, 1000, 1024, 100
    x, y = torch.randn((M * n, p), device="cuda", dtype=torch.bfloat16), torch.arange(M * n, device="cuda", dtype=torch.int32) % C
    gx, gy = torch.randn((4096, 16), device="cuda"), torch.ones(4096, device="cuda")
    s, t = _streams(2)
    results = []
    for together in (False, True):
        soft = B.Context(p, M * n, n, 0.01, 4, model=B.BMGD_SOFTMAX, n_classes=C, barrier_timeout_us=400_000)
        glm = B.Context(16, 4096, 64, 0.01, 4, model=B.BMGD_LOGISTIC, chain=B.BMGD_CHAIN_PERSISTENT, n_workgroups=256, barrier_timeout_us=50_000)
        holder = _Holder(248, 130)
        torch.cuda.synchronize()
        if together:
            holder.start(s)
        glm.run_device_buffer(gx, gy, 4096, s)
        began = torch.cuda.Event(enable_timing=True)
        began.record(t)
        if not together:
            glm.sync()
        soft.run_device_buffer(x, y, M * n, t)
        results.append((glm.get_theta(), soft.get_theta()))
        assert not together or began.elapsed_time(holder.free) > 60
        for c in (soft, glm, holder.ctx):
            c.close()
    for a, b in zip(*results):
        assert np.isfinite(a).all() and np.array_equal(a, b)


def _workspace(p, rows, n, C, T, **limits):
    """A workspace for a softmax context, of zeros, and the arguments that hand it over."""
    import torch
    import paper_2312_08728_amd as B
    cfg = B.bmgd_default_config()
    cfg.p, cfg.buffer_n, cfg.batch_n, cfg.lr, cfg.passes = p, rows, n, 0.01, T
    cfg.model, cfg.n_classes, cfg.x_dtype = B.BMGD_SOFTMAX, C, B.BMGD_BF16
    size = B.bmgd_workspace_bytes(cfg)
    area = torch.zeros(size, dtype=torch.uint8, device="cuda")
    return area, dict(workspace=area, workspace_bytes=size, **limits)


def _came_in_time(area):
    """What meetings of 256 workgroups that were closed before all had come have left in the workspace: how many had (bit 31, their number,
    the tickets drawn by the end; as a float 1e-38 and less, which nothing else there is)."""
    import torch
    words = area[:area.numel() // 4 * 4].view(torch.int32)
    high = (words >> 16) & 0xFFFF
    return (high[(high > 0x8000) & (high < 0x8100) & ((words & 0xFFFF) == 256)] & 0xFF).tolist()


def test_a_short_run_waits_for_units_that_are_free_soon():
    """Forty updates (26 ms by the eight workgroups that find a unit at once, 1 ms by all) behind a kernel that keeps the other units for another
    20 ms."""
    import torch
    import paper_2312_08728_amd as B
    p, C, n = 2048, 1000, 1024
    x, y = torch.randn((10 * n, p), device="cuda", dtype=torch.bfloat16), torch.arange(10 * n, device="cuda", dtype=torch.int32) % C
    s, t = _streams(2)
    area, kw = _workspace(p, 10 * n, n, C, 4)
    holder = _Holder(248, 24)
    with B.Context(p, 10 * n, n, 0.01, 4, model=B.BMGD_SOFTMAX, n_classes=C, **kw) as ctx:
        torch.cuda.synchronize()
        holder.start(s)
        ctx.run_device_buffer(x, y, 10 * n, t)
        ctx.sync()
        assert holder.free.query() and _came_in_time(area) == []
    holder.ctx.close()


@pytest.mark.parametrize("limit", [10, 16, 80])
def test_a_small_limit_on_waits_leaves_an_idle_device_to_all_workgroups(limit):
    """An eighth of 10 to 80 us is less than 256 workgroups may take to arrive."""
    import torch
    import paper_2312_08728_amd as B
    p, C, n = 2048, 1000, 1024
    x, y = torch.randn((n, p), device="cuda", dtype=torch.bfloat16), torch.arange(n, device="cuda", dtype=torch.int32) % C
    area, kw = _workspace(p, n, n, C, 1, barrier_timeout_us=limit)
    closed, s = 0, torch.cuda.Stream()
    with B.Context(p, n, n, 0.01, 1, model=B.BMGD_SOFTMAX, n_classes=C, **kw) as ctx:
        for _ in range(50):
            ctx.run_device_buffer(x, y, n, s)
            ctx.sync()
            closed += len(_came_in_time(area))
    assert closed == 0


@pytest.mark.parametrize("units,limit", [(1, 400_000), (2, 400_000), (7, 400_000), (100, 400_000), (40, 8000), (100, 8000)])
def test_workgroups_that_have_come_share_the_work(units, limit):
    """On the units that a kernel of another context leaves free: some or many items of every phase for each workgroup, dealt unevenly, in
    mini-batches of 1,024 and of 30 rows; the same bits as by all.  A limit of 0.4 s leaves all six updates to one launch, 8 ms one to each.
    (Late workgroups have to be started and leave before a launch ends: where a shader engine has no unit left, once the other kernel has ended.)"""
    import torch
    import paper_2312_08728_amd as B
    p, C, n = 2048, 1000, 1024
    rows = 2 * n + 30
    x, y = torch.randn((rows, p), device="cuda", dtype=torch.bfloat16), torch.arange(rows, device="cuda", dtype=torch.int32) % C
    s, t = _streams(2)
    holder, got = _Holder(256 - units, 150), []
    for together in (False, True):
        area, kw = _workspace(p, rows, n, C, 2, barrier_timeout_us=limit)
        with B.Context(p, rows, n, 0.01, 2, model=B.BMGD_SOFTMAX, n_classes=C, **kw) as ctx:
            torch.cuda.synchronize()
            if together:
                holder.start(s)
            ctx.run_device_buffer(x, y, rows, t)
            got.append(ctx.get_theta())
            assert units < 40 or not (together and holder.free.query())
        assert _came_in_time(area) == ([units] if together else [])
    holder.ctx.close()
    assert np.isfinite(got[0]).all() and np.array_equal(got[0], got[1])


@pytest.mark.parametrize("form", ["fixed partitions", "short buffers", "row subset", "from the host"])
def test_launches_that_go_on_where_the_one_before_ended(form):
    """Five passes by launches of a few updates (a limit of 0.2 ms) and by as few as there can be: the same bits; and the sums of the three
    launches, up to their order and the rounding to bf16 that it decides."""
    import torch
    import paper_2312_08728_amd as B
    w = _case(3000, 1160, 250, 1000, 150, T=5)
    X, y = wl.dataset(w)
    xs, ys = [torch.from_numpy(X[k:k + 1000].view(np.int16)) for k in (0, 1000, 2000)], [torch.from_numpy(y[k:k + 1000]) for k in (0, 1000, 2000)]
    xs, ys = ([v.pin_memory() for v in a] if form == "from the host" else [v.cuda() for v in a] for a in (xs, ys))
    rows = torch.randint(0, 1000, (437,), generator=torch.Generator().manual_seed(1), dtype=torch.int32).cuda()
    s, copy, got = torch.cuda.Stream(), torch.cuda.Stream(), []
    kw = dict(reshuffle=B.BMGD_RESHUFFLE_FIXED, n_buffers=3) if form == "fixed partitions" else {}
    for chain, limit in ((B.BMGD_CHAIN_AUTO, 0), (B.BMGD_CHAIN_AUTO, 200), (B.BMGD_CHAIN_LAUNCH, 0)):
        with B.Context(w.p, 1000, w.n, 0.05, w.T, model=w.model, n_classes=w.C, chain=chain, barrier_timeout_us=limit, **kw) as ctx:
            for xb, yb, short in zip(xs, ys, (7, 149, 151)):
                if form == "from the host":
                    ctx.load_buffer_async(xb, yb, 1000, copy)
                    ctx.run_buffer(s)
                    continue
                if form == "row subset":
                    ctx.set_row_subset(rows, len(rows))
                ctx.run_device_buffer(xb, yb, short if form == "short buffers" else 1000, s)
            got.append(ctx.get_theta())
    assert np.isfinite(got[0]).all() and np.array_equal(got[0], got[1]) and rel_l2(got[0], got[2]) <= 2e-3
