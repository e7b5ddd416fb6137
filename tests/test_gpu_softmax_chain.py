"""The persistent softmax kernel (small mini-batches, 16 classes per workgroup) at the edges of its tiles: class counts around
one, two and more workgroups, rows and features around the tiles of 16 and 32 and the tiles per wavefront, ragged last mini-batches
and a shorter last buffer.  Compared with the fp64 oracle within the bound of the bf16 path (2e-3: bf16 copy of W, bf16
residual; 5e-3 with Adam, which normalises their rounding), and with the three-launch path, whose roundings are the same
up to the order of fp32 sums."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import gpu_run, oracle_run, rel_l2

pytestmark = pytest.mark.gpu


def _case(N, p, C, N0, n, T=2, R=1, alpha=0.05):
    return wl.CONFIGS["cfg5"].scaled(name="case", N=N, p=p, C=C, N0=N0, n=n, T=T, R=R, alpha=alpha)


@pytest.mark.parametrize("N,p,C,N0,n", [
    (70, 8, 2, 40, 1),                 # mini-batches of one row, one feature chunk
    (200, 16, 15, 130, 16),            # one workgroup, not full; one row tile
    (200, 16, 16, 130, 16),            # exactly one workgroup: nothing is exchanged
    (200, 24, 17, 130, 17),            # one class in the second workgroup
    (200, 16, 32, 130, 16),            # exactly two workgroups
    (200, 24, 33, 130, 17),            # one class in the third workgroup
    (600, 128, 64, 400, 128),          # one tile per wavefront both ways, exactly
    (600, 136, 65, 400, 129),          # one more of everything
    (1500, 512, 40, 900, 300),         # several tiles per wavefront
    (2100, 248, 300, 2100, 1024),      # most rows, 19 workgroups: so many classes go to separate launches
    (2100, 248, 250, 2100, 1024),      # most rows that one kernel takes with 16 workgroups
    (900, 1024, 130, 600, 200),        # most features
    (300, 40, 2000, 200, 48),          # 125 workgroups
    (1000, 24, 33, 710, 7),            # 102 updates a pass: the exchange's tags come round; a last mini-batch of 3 rows, a shorter buffer
])
def test_edges(N, p, C, N0, n):
    w = _case(N, p, C, N0, n)
    X, y = wl.dataset(w)
    want = oracle_run(w, X, y)
    got, st = gpu_run(w, X, y)
    assert st.steps == w.steps and np.isfinite(got).all()
    assert rel_l2(got, want) <= 2e-3
    import paper_2312_08728_amd as B
    three, _ = gpu_run(w, X, y, chain=B.BMGD_CHAIN_LAUNCH)
    assert rel_l2(got, three) <= 2e-3


@pytest.mark.parametrize("optimizer", [1, 2, 3])
def test_update_rules_with_a_table_of_rates(optimizer):
    import torch
    import paper_2312_08728_amd as B
    w = _case(1100, 72, 40, 600, 100)
    X, y = wl.dataset(w)
    xd, yd = torch.from_numpy(X.view(np.int16)).cuda(), torch.from_numpy(y).cuda()
    s = torch.cuda.Stream()
    got = []
    for chain in (B.BMGD_CHAIN_AUTO, B.BMGD_CHAIN_LAUNCH):
        ctx = B.Context(w.p, w.N0, w.n, 0.02, w.T, model=w.model, n_classes=w.C, chain=chain, optimizer=optimizer)
        ctx.set_lr_schedule(np.linspace(0.02, 0.002, 9).astype(np.float32))
        for k in range(2):
            lo, hi = wl.buffer_rows(w, k)
            ctx.run_device_buffer(xd[lo:hi], yd[lo:hi], hi - lo, s)
        loss = ctx.eval_loss(xd, yd, w.N, s)                  # reads the bf16 copy the kernel leaves
        got.append((ctx.get_theta(), loss))
        ctx.close()
    assert rel_l2(got[0][0], got[1][0]) <= 5e-3
    assert abs(got[0][1] - got[1][1]) <= 2e-3 * abs(got[1][1])


@pytest.mark.parametrize("optimizer", [1, 2, 3])
@pytest.mark.parametrize("p,n", [(72, 900), (200, 100), (200, 300), (200, 600), (264, 130), (264, 490), (504, 256), (512, 100)])
def test_update_rules_at_every_number_of_tiles(optimizer, p, n):
    """Feature tiles per wavefront 1, 2 (state in registers) and 4 (in memory) beside row tiles 1, 2, 4 and 8, with a ragged mini-batch, a
    shorter second buffer and a third run behind it: the state is carried from launch to launch.  Against the oracle and the launches."""
    import torch
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = _case(5 * n + n // 3, p, 35, 3 * n + 5, n)
    X, y = wl.dataset(w)
    settings = dict(momentum=0.8, beta1=0.9, beta2=0.99, eps=1e-6)
    top = 0.002 if optimizer == 3 else 0.02
    rates = np.linspace(top, top / 10, 13).astype(np.float32)
    ref = O.BMGD(w.model, w.p, w.n, top, w.T, C=w.C)
    ref.set_optimizer(optimizer, **settings)
    ref.set_lr_schedule(rates)
    spans = [wl.buffer_rows(w, k) for k in (0, 1, 0)]
    for lo, hi in spans:
        ref.run_buffer(X[lo:hi], y[lo:hi])
    xd, yd = torch.from_numpy(X.view(np.int16)).cuda(), torch.from_numpy(y).cuda()
    s = torch.cuda.Stream()
    # Adam's first update is alpha times the sign of the gradient, so where the rounding of the residual (2^-9) decides the sign, for
    # about 2^-9 of the coordinates, it is off by twice its size: 2 x 2^-4.5 = 9e-2 of that update, one of 22 here whose
    # rates add up to more than seven times the first one's: 1.2e-2
    bound = 1.2e-2 if optimizer == 3 else 2e-3
    got = []
    for chain in (B.BMGD_CHAIN_AUTO, B.BMGD_CHAIN_LAUNCH):
        ctx = B.Context(w.p, w.N0, w.n, top, w.T, model=w.model, n_classes=w.C, chain=chain, optimizer=optimizer, **settings)
        ctx.set_lr_schedule(rates)
        for lo, hi in spans:
            ctx.run_device_buffer(xd[lo:hi], yd[lo:hi], hi - lo, s)
        got.append(ctx.get_theta().reshape(ref.theta.shape))
        ctx.close()
        assert rel_l2(got[-1], ref.theta) <= bound, chain
    assert rel_l2(got[0], got[1]) <= bound


@pytest.mark.parametrize("bad,C", [(np.inf, 40), (-np.inf, 40), (np.nan, 40), (np.inf, 20), (np.nan, 20),
                                   (np.inf, 16), (-np.inf, 10), (np.nan, 16), (np.nan, 17), (np.inf, 130)])
def test_values_that_are_not_finite_spread_as_in_three_launches(bad, C):
    import torch
    import paper_2312_08728_amd as B
    w = _case(64, 32, C, 64, 64, T=1)
    X, y = wl.dataset(w)
    x = torch.from_numpy(X.view(np.int16)).view(torch.bfloat16).cuda()
    x[5, 3] = float(bad)
    yd = torch.from_numpy(y).cuda()
    w0 = (np.random.default_rng(0).standard_normal((w.p, C)) * 0.1).astype(np.float32)
    got = []
    for chain in (B.BMGD_CHAIN_AUTO, B.BMGD_CHAIN_LAUNCH):
        ctx = B.Context(w.p, 64, 64, 0.05, 1, model=w.model, n_classes=C, chain=chain)
        ctx.set_theta(w0)
        ctx.run_device_buffer(x, yd, 64, torch.cuda.Stream())
        got.append(ctx.get_theta())
        ctx.close()
    assert np.array_equal(np.isnan(got[0]), np.isnan(got[1]))


def test_row_subset_and_fixed_partitions():
    import torch
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = _case(900, 64, 40, 900, 100, T=3)
    X, y = wl.dataset(w)
    sel = np.random.default_rng(3).permutation(900)[:430].astype(np.int32)
    ref = O.BMGD(w.model, w.p, w.n, w.alpha, w.T, C=w.C, reshuffle=O.FIXED, K_fixed=1)
    ref.run_buffer(X[sel], y[sel])
    ref.run_buffer(X, y)
    ctx = B.Context(w.p, w.N0, w.n, w.alpha, w.T, model=w.model, n_classes=w.C, reshuffle=B.BMGD_RESHUFFLE_FIXED, n_buffers=1)
    xd, yd, sd = torch.from_numpy(X.view(np.int16)).cuda(), torch.from_numpy(y).cuda(), torch.from_numpy(sel).cuda()
    s = torch.cuda.Stream()
    ctx.set_row_subset(sd, len(sel))
    ctx.run_device_buffer(xd, yd, 900, s)
    ctx.run_device_buffer(xd, yd, 900, s)
    got = ctx.get_theta().reshape(ref.theta.shape)
    ctx.close()
    assert rel_l2(got, ref.theta) <= 2e-3


@pytest.mark.parametrize("N,p,C,N0,n,optimizer", [
    (70, 8, 17, 40, 1, 0),             # one row, one feature chunk, one class in the second workgroup
    (1000, 24, 33, 710, 7, 0),         # more updates a pass than the exchange has tags
    (1000, 200, 130, 700, 100, 0),     # ragged mini-batches, a shorter second buffer
    (900, 264, 40, 500, 130, 1),       # state in memory
    (900, 200, 300, 500, 100, 2),
    (900, 72, 33, 500, 300, 3),
    (1300, 200, 100, 700, 600, 0),     # more than 512 rows: two to a thread of the exchange
    (400, 1024, 2000, 200, 64, 0),     # most features, 125 workgroups
])
def test_one_workgroup_makes_the_pass_where_the_others_do_not_come(N, p, C, N0, n, optimizer):
    """With a limit on waits that leaves no time to meet, one workgroup makes every pass alone: the same sums in the same order, so
    the same W (and state: two buffers, and a run behind them) bit for bit with all rules but Adam's, and no error."""
    import torch
    import paper_2312_08728_amd as B
    w = _case(N, p, C, N0, n)
    X, y = wl.dataset(w)
    xd, yd = torch.from_numpy(X.view(np.int16)).cuda(), torch.from_numpy(y).cuda()
    s = torch.cuda.Stream()
    got = []
    for limit in (0, 1):
        ctx = B.Context(w.p, w.N0, w.n, 0.01, w.T, model=w.model, n_classes=w.C, optimizer=optimizer, barrier_timeout_us=limit)
        ctx.set_lr_schedule(np.linspace(0.02, 0.002, 9).astype(np.float32))
        for k in (0, 1, 0):
            lo, hi = wl.buffer_rows(w, k)
            ctx.run_device_buffer(xd[lo:hi], yd[lo:hi], hi - lo, s)
        got.append((ctx.get_theta(), ctx.eval_loss(xd, yd, w.N, s)))
        ctx.close()
    assert np.isfinite(got[0][0]).all() and got[0][0].any()
    if optimizer == 3:
        # Adam's products may be joined into multiply-adds differently in the two places: a last bit (2^-24) per update, which
        # takes a value's bf16 copy to its neighbour (2^-8) once in 2^15 times: 2^-8 2^-7.5 = 2e-5 of the copy, rms
        assert rel_l2(got[1][0], got[0][0]) <= 1e-4 and abs(got[1][1] - got[0][1]) <= 1e-4 * got[0][1]
    else:
        assert np.array_equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]


def test_contexts_that_compete_for_the_compute_units():
    """Softmax runs of several contexts and a long run of the persistent logistic kernel (one workgroup to a compute unit), all on
    streams of their own: whichever workgroups find room, every run ends as it does with the device to itself."""
    import torch
    import paper_2312_08728_amd as B
    w = _case(4000, 256, 2000, 4000, 500)
    X, y = wl.dataset(w)
    xd, yd = torch.from_numpy(X.view(np.int16)).cuda(), torch.from_numpy(y).cuda()
    v = wl.CONFIGS["cfg3"].scaled(name="other", N=200_000, p=200, N0=200_000, n=4096, T=4, R=1)
    VX, vy = wl.dataset(v)
    vx, vyd = torch.from_numpy(VX).cuda(), torch.from_numpy(vy).cuda()
    streams = [torch.cuda.Stream() for _ in range(3)]

    def contexts():
        return [B.Context(w.p, w.N0, w.n, w.alpha, w.T, model=w.model, n_classes=w.C, seed=i) for i in range(2)], \
               B.Context(v.p, v.N0, v.n, v.alpha, v.T, model=v.model, chain=B.BMGD_CHAIN_PERSISTENT)

    results = []
    for together in (False, True):
        soft, glm = contexts()
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


@pytest.mark.parametrize("optimizer", [0, 1, 3])
@pytest.mark.parametrize("bad,C", [(np.inf, 10), (np.nan, 10), (-np.inf, 33), (np.nan, 130)])
def test_a_new_estimate_ends_what_values_that_are_not_finite_left_behind(bad, C, optimizer):
    """Classes that only fill up the last workgroup stay zero whatever the rows hold: after bmgd_set_theta a run over clean rows
    is the run of a new context."""
    import torch
    import paper_2312_08728_amd as B
    w = _case(128, 40, C, 128, 64)
    X, y = wl.dataset(w)
    clean = torch.from_numpy(X.view(np.int16)).view(torch.bfloat16).cuda()
    x = clean.clone()
    x[5, 3] = float(bad)
    yd, s = torch.from_numpy(y).cuda(), torch.cuda.Stream()
    w0 = (np.random.default_rng(0).standard_normal((w.p, C)) * 0.1).astype(np.float32)
    got = []
    for first in (x, None):
        ctx = B.Context(w.p, 128, 64, 0.02, 1, model=w.model, n_classes=C, optimizer=optimizer)
        if first is not None:
            ctx.set_theta(w0)
            ctx.run_device_buffer(first, yd, 128, s)
            assert np.isnan(ctx.get_theta()).any()
            ctx.reset_optimizer()
            ctx.set_position(0)
        ctx.set_theta(w0)
        ctx.run_device_buffer(clean, yd, 128, s)
        got.append(ctx.get_theta())
        ctx.close()
    assert np.isfinite(got[0]).all() and np.array_equal(got[0], got[1])


def test_rows_that_are_all_but_certain_keep_their_residual():
    """P - 1 of a class whose logit stands 12 above all others, at logits of 340: 1.2e-4, which a normaliser kept as one fp32
    number of that size (spacing 3e-5) would lose.  The residual is rounded to bf16 (2^-9 of it), 1 - P to fp32 (2^-24, 2^-11 of
    the difference): 2^-8 in all."""
    import torch
    import paper_2312_08728_amd as B
    n, p, C = 64, 8, 20
    gen = torch.Generator().manual_seed(1)
    x = torch.zeros((n, p))
    x[:, 0] = 1.0
    x[:, 1:] = torch.rand((n, p - 1), generator=gen) + 0.5
    x = x.bfloat16()
    w0 = np.zeros((p, C), dtype=np.float32)
    w0[0], w0[0, 0] = 328.0, 340.0                         # exact in bf16
    prob = torch.softmax(torch.from_numpy(w0[0]).double(), 0)
    prob[0] = -prob[1:].sum()                              # the residual of class 0, the label of every row
    want = -0.5 * x.double().mean(0)[1:, None] * prob[None, :]
    for chain in (B.BMGD_CHAIN_AUTO, B.BMGD_CHAIN_LAUNCH):
        ctx = B.Context(p, n, n, 0.5, 1, model=B.BMGD_SOFTMAX, n_classes=C, chain=chain)
        ctx.set_theta(w0)
        ctx.run_device_buffer(x.cuda(), torch.zeros(n, dtype=torch.int32, device="cuda"), n, None)
        got = ctx.get_theta()[1:]
        ctx.close()
        assert np.abs(got / want.numpy() - 1.0).max() <= 2.0 ** -8, chain


def test_a_workspace_of_the_size_that_separate_launches_need_is_taken():
    """Its size without the mini-batches in operand order and the exchange: then another kernel makes the updates."""
    import torch
    import paper_2312_08728_amd as B
    w = _case(900, 8, 20, 900, 16)
    X, y = wl.dataset(w)
    cfg = B.bmgd_default_config()
    cfg.p, cfg.buffer_n, cfg.batch_n, cfg.lr, cfg.passes = w.p, w.N0, w.n, w.alpha, w.T
    cfg.model, cfg.n_classes, cfg.x_dtype, cfg.chain = B.BMGD_SOFTMAX, w.C, B.BMGD_BF16, B.BMGD_CHAIN_LAUNCH
    size = B.bmgd_workspace_bytes(cfg)
    cfg.chain = B.BMGD_CHAIN_AUTO
    assert size < B.bmgd_workspace_bytes(cfg)
    area = torch.zeros(size, dtype=torch.uint8, device="cuda")
    got, _ = gpu_run(w, X, y, workspace=area, workspace_bytes=size)
    assert rel_l2(got, oracle_run(w, X, y)) <= 2e-3
    with pytest.raises(B.BmgdError) as e:
        gpu_run(w, X, y, workspace=area, workspace_bytes=size - 256)
    assert e.value.code == B.BMGD_ENOMEM


@pytest.mark.parametrize("size", [30.0, 1e4, 1e7, 1e20, 2e38])
def test_logits_of_any_size(size):
    """Logits of -size, 0 and size in turn over the classes of three workgroups: the classes at the top share each row alike, up to the
    rounding of the residual to bf16 (2^-9) and of the fp32 update (2^-24 of it per row): 2^-8."""
    import torch
    import paper_2312_08728_amd as B
    n, p, C = 40, 8, 37
    x = torch.zeros((n, p))
    x[:, 0] = 1.0
    x[:, 1:] = torch.rand((n, p - 1), generator=torch.Generator().manual_seed(2)) + 0.5
    x = x.bfloat16()
    w0 = np.zeros((p, C), dtype=np.float32)
    w0[0] = torch.tensor([size * (c % 3 - 1) for c in range(C)]).bfloat16().float().numpy()
    prob = torch.softmax(torch.from_numpy(w0[0]).double(), 0)
    prob[2] -= 1.0                                         # every row's label
    want = (-0.5 * x.double().mean(0)[1:, None] * prob[None, :]).numpy()
    for limit in (0, 1):                                   # (1: by one workgroup alone)
        ctx = B.Context(p, n, n, 0.5, 1, model=B.BMGD_SOFTMAX, n_classes=C, barrier_timeout_us=limit)
        ctx.set_theta(w0)
        ctx.run_device_buffer(x.cuda(), torch.full((n,), 2, dtype=torch.int32, device="cuda"), n, None)
        got = ctx.get_theta()[1:]
        ctx.close()
        assert np.abs(got - want).max() <= 2.0 ** -8 * np.abs(want).max()
        some = np.abs(want) > 1e-12
        assert np.abs(got[some] / want[some] - 1.0).max() <= 2.0 ** -8 and np.abs(got[~some]).max(initial=0.0) <= 1e-12
