"""The persistent kernel for rows of up to 1024 floats whose share of a step fits the registers (eight row wavefronts
with two alternating groups of rows, four exchange wavefronts): every register shape it is built for, against the oracle."""
import numpy as np
import pytest

import workloads as wl
import gpu_util as U
from gpu_util import gpu_run, oracle_run, rel_l2, coord_err

pytestmark = pytest.mark.gpu

TOL = 1e-4
NARROW_THREADS = 768          # 12 wavefronts


def _case(model, N, p, N0, n, T, R, alpha):
    base = wl.CONFIGS["cfg3" if model == wl.LOGISTIC else "cfg2"]
    return base.scaled(name="case", N=N, p=p, N0=N0, n=n, T=T, R=R, alpha=alpha, x_cov="identity")


# (model, p, n, G, N0): floats per load V, chunks per lane CPL, rows per lane slot PF, lanes per row L that result
SHAPES = [
    (wl.LOGISTIC, 200, 4096, 256, 10_000),   # V 4, CPL 1, PF 2, L 64: cfg3's shape; a short last mini-batch; 9 steps per launch (odd)
    (wl.LINEAR, 100, 1000, 64, 6_000),       # V 4, CPL 1, PF 1, L 32: two rows side by side in a wavefront
    (wl.LINEAR, 36, 5000, 128, 12_000),      # V 4, CPL 1, PF 2, L 16: four rows side by side
    (wl.LOGISTIC, 1024, 2048, 256, 5_000),   # V 4, CPL 4, PF 1: the widest rows
    (wl.LINEAR, 512, 4096, 256, 9_000),      # V 4, CPL 2, PF 2
    (wl.LINEAR, 250, 3000, 128, 7_000),      # V 2, CPL 2, PF 4
    (wl.LOGISTIC, 70, 8000, 128, 17_000),    # V 2, CPL 1, PF 8: the most rows per lane slot
    (wl.LINEAR, 600, 128, 8, 1_000),         # V 4, CPL 4, PF 2 on the fewest workgroups
    (wl.LOGISTIC, 200, 1400, 24, 5_000),     # V 4, CPL 1, PF 8 on 24 workgroups: 32 floats of rows per lane and group
]


@pytest.mark.parametrize("model,p,n,G,N0", SHAPES)
def test_register_shapes_against_the_oracle(model, p, n, G, N0):
    import paper_2312_08728_amd as B
    w = _case(model, 2 * N0 - 77, p, N0, n, T=3, R=2, alpha=0.5 / (p + 10) if model == wl.LINEAR else 0.1)
    X, y = wl.dataset(w)
    want = oracle_run(w, X, y)
    got, st = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT)
    assert st.threads_per_group == NARROW_THREADS and st.n_workgroups == G, (st.threads_per_group, st.n_workgroups)
    assert st.launched[2:4] == (U.NARROW, U.TWO_TRIPS if G <= 24 else U.BY_DIE)
    assert st.steps == w.steps
    assert rel_l2(got, want) <= TOL and coord_err(got, want) <= 10 * TOL


@pytest.mark.parametrize("optimizer", [1, 2, 3])
def test_update_rules_with_state(optimizer):
    """Momentum, NAG and Adam keep their state per coordinate in global memory; the first exchange wavefront of the
    workgroup that owns a slice updates it."""
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = _case(wl.LOGISTIC, 12_000, 200, 6_000, 2048, T=2, R=2, alpha=0.01 if optimizer == 3 else 0.05)
    X, y = wl.dataset(w)
    ref = O.BMGD(w.model, w.p, w.n, w.alpha, w.T)
    ref.set_optimizer(optimizer)
    for _ in range(w.R):
        for k in range(2):
            ref.run_buffer(X[k * 6000:(k + 1) * 6000], y[k * 6000:(k + 1) * 6000])
    got, st = gpu_run(w, X, y, n_workgroups=64, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer)
    assert st.threads_per_group == NARROW_THREADS
    assert rel_l2(got, ref.theta) <= TOL


def test_is_reproducible_and_equals_the_loader_path():
    import paper_2312_08728_amd as B
    w = _case(wl.LOGISTIC, 30_000, 200, 10_000, 4096, T=2, R=2, alpha=0.1)
    X, y = wl.dataset(w)
    a, sa = gpu_run(w, X, y, chain=B.BMGD_CHAIN_PERSISTENT)
    b, _ = gpu_run(w, X, y, chain=B.BMGD_CHAIN_PERSISTENT, resident=True)
    c, _ = gpu_run(w, X, y, chain=B.BMGD_CHAIN_PERSISTENT)
    assert sa.threads_per_group == NARROW_THREADS
    assert np.array_equal(a, b) and np.array_equal(a, c)


def test_other_kernels_keep_their_cases():
    """Few workgroups or sums few enough for every workgroup to add up itself: one trip; odd p: twelve row wavefronts; steps that do not fit
    the registers, and wide rows on few workgroups: the general kernel.  (1024 threads, 512 for the last.)"""
    import paper_2312_08728_amd as B
    for kw, p, n, N0, launched in ((dict(n_workgroups=4), 200, 1000, 4000, (U.GENERAL, U.ONE_TRIP)),      # 1000 rows on 48 row slots
                                   (dict(n_workgroups=4), 200, 130, 1000, (U.NARROW, U.ONE_TRIP)),        # fewer than eight workgroups
                                   (dict(n_workgroups=16), 100, 1000, 4000, (U.NARROW, U.ONE_TRIP)),      # 16 * 100 words
                                   (dict(n_workgroups=64), 201, 1000, 4000, (U.NARROW, U.BY_DIE)),        # odd p
                                   (dict(n_workgroups=8), 200, 4096, 9000, (U.GENERAL, U.ONE_TRIP)),      # 64 slots: 64 rows per slot
                                   (dict(n_workgroups=32), 200, 4096, 9000, (U.GENERAL, U.TWO_TRIPS)),
                                   (dict(n_workgroups=8), 1026, 300, 700, (U.GENERAL, U.TWO_TRIPS))):     # 38 rows of more than 1024 floats each
        w = _case(wl.LINEAR, 2 * N0, p, N0, n, T=2, R=1, alpha=0.5 / (p + 10))
        X, y = wl.dataset(w)
        want = oracle_run(w, X, y)
        got, st = gpu_run(w, X, y, chain=B.BMGD_CHAIN_PERSISTENT, **kw)
        assert st.threads_per_group == (1024 if p <= 1024 else 512), (kw, p, st.threads_per_group)
        assert st.launched[2:4] == launched, (kw, p, st.launched)
        assert rel_l2(got, want) <= TOL


def test_more_passes_than_one_launch_holds_and_a_rate_per_update():
    """Five passes are two launches (four passes, then one): tags, versions and the position in the table of learning
    rates carry over from launch to launch."""
    import torch
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = _case(wl.LOGISTIC, 12_000, 200, 6_000, 2048, T=5, R=1, alpha=0.1)
    X, y = wl.dataset(w)
    steps = 2 * 5 * 3
    sched = (0.1 * (0.5 + 0.5 * np.cos(np.pi * np.arange(steps) / steps))).astype(np.float32)
    ref = O.BMGD(w.model, w.p, w.n, w.alpha, w.T)
    ref.set_lr_schedule(sched)
    ctx = B.Context(w.p, w.N0, w.n, w.alpha, w.T, model=w.model, n_workgroups=64, chain=B.BMGD_CHAIN_PERSISTENT)
    ctx.set_lr_schedule(sched)
    xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    s = torch.cuda.Stream()
    for k in range(2):
        ref.run_buffer(X[k * 6000:(k + 1) * 6000], y[k * 6000:(k + 1) * 6000])
        ctx.run_device_buffer(xd[k * 6000:(k + 1) * 6000], yd[k * 6000:(k + 1) * 6000], 6000, s)
    got = ctx.get_theta()
    st = ctx.stats()
    ctx.close()
    assert st.threads_per_group == NARROW_THREADS and st.steps == steps and st.chain_launches == 4
    assert rel_l2(got, ref.theta) <= TOL


# (model, p, n, G, N0): the form with one trip over the fabric per step (G p <= 4096: twelve row wavefronts, 1024 threads), and odd rows
# over two levels.  Columns travel as pairs, 8 to 64 of them to an exchange wavefront, and 64 / (pairs) workgroups side by side.
ONE_TRIP = [
    (wl.LOGISTIC, 1, 40, 1, 500),        # one column, one workgroup: no exchange
    (wl.LOGISTIC, 2, 300, 3, 1_000),     # one pair; fewer workgroups than lane groups (8)
    (wl.LINEAR, 15, 500, 7, 1_700),      # eight pairs, one with a place that stands for no column; 7 of 8 lane groups
    (wl.LOGISTIC, 16, 900, 9, 2_000),    # 9 workgroups in groups of 8: the second load repeats seven
    (wl.LINEAR, 17, 2000, 33, 5_000),    # two wavefronts have columns; five loads a lane, the last repeats seven workgroups; odd G
    (wl.LOGISTIC, 64, 700, 11, 2_100),   # 32 pairs, eight lane groups: the second load repeats five
    (wl.LINEAR, 65, 1200, 63, 3_000),    # 34 pairs, sixteen to a wavefront; 16 loads per lane, in two rounds
    (wl.LOGISTIC, 123, 777, 32, 3_000),  # 62 pairs
    (wl.LOGISTIC, 128, 1024, 32, 3_000), # 64: sixteen to each wavefront
    (wl.LINEAR, 129, 600, 31, 2_000),    # 66, 32 to a wavefront: the third has two, the last none
    (wl.LOGISTIC, 255, 300, 16, 1_000),  # 128, one with a place that stands for no column
    (wl.LINEAR, 256, 350, 16, 1_000),    # 32 to each wavefront
    (wl.LOGISTIC, 258, 200, 15, 700),    # 130, 64 to a wavefront: the third has two, the last none
    (wl.LOGISTIC, 512, 90, 8, 400),      # the widest rows
    (wl.LOGISTIC, 201, 1500, 64, 4_000), # odd rows over two levels
    (wl.LINEAR, 33, 4000, 128, 9_000),   # odd rows over two levels, four rows side by side in a wavefront
]


@pytest.mark.parametrize("optimizer", [0, 1, 3])
@pytest.mark.parametrize("model,p,n,G,N0", ONE_TRIP)
def test_one_trip_and_odd_rows_against_the_oracle(model, p, n, G, N0, optimizer):
    """Three launches of theta, state and tags carried over (two buffers, the second run with five passes as two launches)."""
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = _case(model, 2 * N0 - 77, p, N0, n, T=5, R=1, alpha=0.01 if optimizer == 3 else 0.05 if model == wl.LOGISTIC else 0.2 / (p + 10))
    X, y = wl.dataset(w)
    ref = O.BMGD(w.model, w.p, w.n, w.alpha, w.T)
    if optimizer:
        ref.set_optimizer(optimizer)
    for k in range(2):
        ref.run_buffer(X[k * N0:(k + 1) * N0], y[k * N0:(k + 1) * N0])
    got, st = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer)
    assert st.threads_per_group == 1024 and st.n_workgroups == G, (st.threads_per_group, st.n_workgroups)
    assert st.launched[2:4] == (U.NARROW, U.ONE_TRIP if G * p <= 4096 else U.BY_DIE)
    assert rel_l2(got, ref.theta) <= TOL
    again, _ = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer, resident=True)
    assert np.array_equal(got, again)


@pytest.mark.parametrize("p,n,launched", [(16, 768, 4), (30, 384, 4), (64, 96, 2), (15, 96, 1)])
def test_one_workgroup_is_chosen_for_the_chain_kernel_alone(p, n, launched):
    """Shapes whose step one workgroup of the chain's kernel holds: steps launched one by one keep 12 KB of rows a workgroup."""
    import paper_2312_08728_amd as B
    w = _case(wl.LOGISTIC, 3 * n, p, 2 * n, n, T=2, R=1, alpha=0.05)
    X, y = wl.dataset(w)
    want = oracle_run(w, X, y)
    for chain, G in ((B.BMGD_CHAIN_PERSISTENT, 1), (B.BMGD_CHAIN_LAUNCH, launched)):
        got, st = gpu_run(w, X, y, chain=chain)
        assert st.chain == chain and st.n_workgroups == G
        assert rel_l2(got, want) <= TOL


# (model, p, n, G, N0): sums added up over two levels, on the dies first.  A line of 16 columns belongs to one wavefront of one workgroup of each
# die (four take part, three for rows of more than 1024 floats, which may have two lines), which asks for four workgroups' words a lane.
BY_DIE = [
    (wl.LINEAR, 10, 3000, 136, 7_000),       # one line; 17 workgroups a die
    (wl.LOGISTIC, 16, 4000, 256, 9_000),     # a full line
    (wl.LOGISTIC, 20, 9000, 256, 20_000),    # two lines, the second of four columns; 32 workgroups a die
    (wl.LINEAR, 128, 900, 40, 3_000),        # 5 workgroups a die: fewer than a wavefront has groups of lanes
    (wl.LOGISTIC, 500, 700, 64, 2_000),      # 8 a die, 32 lines: every wavefront has one
    (wl.LINEAR, 200, 1500, 72, 4_000),       # 9 a die: the second load repeats seven
    (wl.LOGISTIC, 1024, 600, 128, 2_000),    # 64 lines for 64 wavefronts
    (wl.LINEAR, 300, 2400, 200, 6_000),      # 25 a die
    (wl.LOGISTIC, 1028, 500, 88, 1_500),     # 65 lines for 33 wavefronts, two each but one
    (wl.LINEAR, 2048, 400, 176, 1_000),      # 128 for 66
    (wl.LOGISTIC, 1500, 900, 256, 2_500),    # 94 for 96: the second line of each is beyond the end
    (wl.LINEAR, 2052, 300, 168, 900),        # 129 lines for 63 wavefronts, up to three each
    (wl.LOGISTIC, 4096, 250, 256, 600),      # 256 for 96
]


@pytest.mark.parametrize("optimizer", [0, 2, 3])
@pytest.mark.parametrize("model,p,n,G,N0", BY_DIE)
def test_sums_added_up_on_the_dies_first(model, p, n, G, N0, optimizer):
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = _case(model, 2 * N0 - 77, p, N0, n, T=5, R=1, alpha=0.01 if optimizer == 3 else 0.05 if model == wl.LOGISTIC else 0.2 / (p + 10))
    X, y = wl.dataset(w)
    ref = O.BMGD(w.model, w.p, w.n, w.alpha, w.T)
    if optimizer:
        ref.set_optimizer(optimizer)
    for k in range(2):
        ref.run_buffer(X[k * N0:(k + 1) * N0], y[k * N0:(k + 1) * N0])
    got, st = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer)
    assert st.launched[:4] == (G, *((704, U.SPLIT) if p > 1024 else (NARROW_THREADS, U.NARROW)), U.BY_DIE)
    assert rel_l2(got, ref.theta) <= TOL
    again, _ = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer, resident=True)
    assert np.array_equal(got, again)
    # words at device scope, as where the workgroups of a die are on several: the same sums in the same order
    far, _ = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer, far=True)
    assert np.array_equal(got, far)


# (p, batch, G, rows of the short buffer): mini-batches of a full buffer in two trips, a short one's over two levels
BOTH = [(1030, 1_200, 96, 1_000), (2044, 2_200, 176, 2_100), (3000, 600, 256, 500)]


@pytest.mark.parametrize("optimizer", [0, 1, 3])
@pytest.mark.parametrize("p,n,G,short", BOTH)
def test_runs_of_a_context_that_exchange_in_both_ways(p, n, G, short, optimizer):
    """Tags, words, theta and the state of an update rule go from one to the other and back."""
    import torch
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    N0 = 2 * n + 77
    w = _case(wl.LOGISTIC, 3 * N0, p, N0, n, T=2, R=1, alpha=0.01 if optimizer == 3 else 0.05)
    X, y = wl.dataset(w)
    ref = O.BMGD(w.model, w.p, w.n, w.alpha, w.T)
    if optimizer:
        ref.set_optimizer(optimizer)
    ctx = B.Context(w.p, w.N0, w.n, w.alpha, w.T, model=w.model, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer)
    s = torch.cuda.Stream()
    assert U.launched(ctx, n)[:4] == (G, 704, U.SPLIT, U.TWO_TRIPS) and U.launched(ctx, short)[3] == U.BY_DIE
    for k, rows in enumerate((N0, short, N0, short, short)):
        lo = k % 3 * N0
        xb, yb = np.ascontiguousarray(X[lo:lo + rows]), np.ascontiguousarray(y[lo:lo + rows])
        ref.run_buffer(xb, yb)
        xd, yd = torch.from_numpy(xb).cuda(), torch.from_numpy(yb).cuda()
        ctx.run_device_buffer(xd, yd, rows, s)
        assert rel_l2(ctx.get_theta(), ref.theta) <= TOL, (k, rows)
    ctx.close()


# (model, p, n, G, N0): rows whose length is no multiple of four floats, taken as vectors of four of which the last starts four columns before
# the row's end and repeats one to three columns.
ANY_LENGTH = [
    (wl.LOGISTIC, 9, 300, 2, 700),        # three vectors, the last repeats three columns; one trip
    (wl.LINEAR, 10, 900, 5, 2_000),       # two
    (wl.LOGISTIC, 11, 700, 3, 2_000),     # one
    (wl.LINEAR, 61, 500, 12, 1_500),      # the last line of 16 holds one vector of which one column counts
    (wl.LOGISTIC, 129, 300, 8, 900),      # 33 vectors: a lane's second half is empty
    (wl.LINEAR, 257, 200, 8, 600),        # 65 vectors: the second of a lane but one
    (wl.LOGISTIC, 511, 250, 8, 700),      # the widest odd rows of one trip, three rows a lane
    (wl.LINEAR, 62, 6000, 128, 14_000),   # sums over two levels
    (wl.LOGISTIC, 302, 1000, 96, 3_000),
    (wl.LINEAR, 513, 700, 80, 2_000),     # four vectors a lane, three of them empty but for one lane
    (wl.LOGISTIC, 1023, 500, 128, 1_500),
    (wl.LINEAR, 1022, 100, 16, 400),      # two trips
    (wl.LOGISTIC, 1026, 300, 64, 900),    # rows split over the wavefronts: in two trips
    (wl.LINEAR, 1030, 500, 96, 1_500),    # and over two levels
    (wl.LOGISTIC, 2046, 600, 256, 1_500),
]


@pytest.mark.parametrize("optimizer", [0, 1, 3])
@pytest.mark.parametrize("model,p,n,G,N0", ANY_LENGTH)
def test_rows_of_any_length(model, p, n, G, N0, optimizer):
    """Two buffers of five passes (two launches each): theta and state carry over by position."""
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = _case(model, 2 * N0 - 77, p, N0, n, T=5, R=1, alpha=0.01 if optimizer == 3 else 0.05 if model == wl.LOGISTIC else 0.2 / (p + 10))
    X, y = wl.dataset(w)
    ref = O.BMGD(w.model, w.p, w.n, w.alpha, w.T)
    if optimizer:
        ref.set_optimizer(optimizer)
    for k in range(2):
        ref.run_buffer(X[k * N0:(k + 1) * N0], y[k * N0:(k + 1) * N0])
    got, st = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer)
    assert st.launched[:3] == (G, *((704, U.SPLIT) if p > 1024 else (1024 if G * p <= 4096 else NARROW_THREADS, U.NARROW)))
    assert st.launched[3] == (U.ONE_TRIP if G * p <= 4096 else U.TWO_TRIPS if p in (1022, 1026) else U.BY_DIE)
    assert rel_l2(got, ref.theta) <= TOL and coord_err(got, ref.theta) <= 10 * TOL
    again, _ = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer, resident=True)
    assert np.array_equal(got, again)


@pytest.mark.parametrize("p,n,G,threads", [(65, 1152, 16, 1024), (128, 1536, 16, 1024), (128, 1537, 32, 1024), (64, 1200, 25, 1024), (200, 192, 8, 1024), (200, 193, 16, 1024), (256, 768, 16, 1024), (256, 769, 64, NARROW_THREADS),
                                           (400, 96, 4, 1024), (401, 97, 8, 1024), (512, 288, 8, 1024), (300, 289, 24, NARROW_THREADS)])
def test_workgroups_chosen_for_rows_of_65_to_512_floats(p, n, G, threads):
    """As few as let every workgroup add up all sums, where they hold the rows."""
    import paper_2312_08728_amd as B
    w = _case(wl.LOGISTIC, 4 * n, p, 2 * n + 5, n, T=2, R=1, alpha=0.05)
    X, y = wl.dataset(w)
    got, st = gpu_run(w, X, y, chain=B.BMGD_CHAIN_PERSISTENT)
    assert (st.n_workgroups, st.threads_per_group, st.launched[2]) == (G, threads, U.NARROW)
    assert st.launched[3] == (U.ONE_TRIP if threads == 1024 else U.TWO_TRIPS if p == 300 else U.BY_DIE)
    assert rel_l2(got, oracle_run(w, X, y)) <= TOL


# (model, p, n, G, N0): one trip with few columns on more than 64 workgroups: two or four pairs to an exchange wavefront, of which the last may have
# none, and up to eight words a lane; beyond 128 workgroups nine to sixteen columns go over two levels if the workgroups are whole eights.
FEW_COLUMNS = [
    (wl.LOGISTIC, 3, 900, 100, 2_000),     # two pairs: one wavefront has columns
    (wl.LINEAR, 5, 2_000, 255, 4_500),     # three pairs: two; eight words a lane, the last loads repeat one workgroup
    (wl.LOGISTIC, 8, 1_500, 200, 3_500),   # vectors of four
    (wl.LOGISTIC, 11, 1_200, 131, 2_500),  # eight words a lane; with state four pairs a wavefront, in two rounds
    (wl.LINEAR, 13, 1_500, 128, 3_500),    # four words a lane; the last pair has no column but a place
    (wl.LOGISTIC, 16, 800, 66, 1_900),     # three words a lane
    (wl.LOGISTIC, 16, 800, 64, 1_900),     # eight pairs: one wavefront, eight words a lane
    (wl.LINEAR, 17, 1_200, 65, 3_000),     # four pairs: nine of them, three wavefronts
    (wl.LOGISTIC, 32, 1_500, 128, 3_500),  # eight words a lane
    (wl.LINEAR, 33, 1_000, 80, 2_500),     # eight pairs
]


@pytest.mark.parametrize("optimizer", [0, 1, 3])
@pytest.mark.parametrize("model,p,n,G,N0", FEW_COLUMNS)
def test_few_columns_on_many_workgroups(model, p, n, G, N0, optimizer):
    import paper_2312_08728_amd as B
    from oracle import bmgd as O
    w = _case(model, 2 * N0 - 77, p, N0, n, T=5, R=1, alpha=0.01 if optimizer == 3 else 0.05 if model == wl.LOGISTIC else 0.2 / (p + 10))
    X, y = wl.dataset(w)
    ref = O.BMGD(w.model, w.p, w.n, w.alpha, w.T)
    if optimizer:
        ref.set_optimizer(optimizer)
    for k in range(2):
        ref.run_buffer(X[k * N0:(k + 1) * N0], y[k * N0:(k + 1) * N0])
    got, st = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer)
    assert st.launched[:4] == (G, 1024, U.NARROW, U.ONE_TRIP)
    assert rel_l2(got, ref.theta) <= TOL
    again, _ = gpu_run(w, X, y, n_workgroups=G, chain=B.BMGD_CHAIN_PERSISTENT, optimizer=optimizer, resident=True)
    assert np.array_equal(got, again)
