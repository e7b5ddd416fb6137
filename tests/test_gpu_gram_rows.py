"""The moment matrices of 96 features and more with every wavefront on its own rows (many mini-batches, or few long ones over two workgroups):
tile, row-share and operand edges.  fp32 sums, as in the other tests of this form: 1e-4 against the oracle."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import gpu_run, oracle_run, rel_l2

pytestmark = pytest.mark.gpu


def _case(p, N0, n, T=2):
    return wl.CONFIGS["cfg2"].scaled(name="case", N=2 * N0 - 5, p=p, N0=N0, n=n, T=T, R=1, alpha=0.1 / (p + 10), x_cov="identity")


@pytest.mark.parametrize("chain", [3, 5])            # the chain's layout, and dense for the products
# one workgroup by rows, and two; a last mini-batch of 3 rows (at p = 97, 111 and 128 the first is for the staged kernel, at p = 128 the second too)
@pytest.mark.parametrize("M,n", [(85, 601), (7, 2003), (105, 601), (7, 8003)])
@pytest.mark.parametrize("p", [96, 97, 100, 111, 112, 127, 128])
def test_tile_edges_against_the_oracle(p, M, n, chain):
    w = _case(p, M * n + 3, n)
    X, y = wl.dataset(w)
    got, st = gpu_run(w, X, y, chain=chain)
    assert st.chain == chain and rel_l2(got, oracle_run(w, X, y)) <= 1e-4
    again, _ = gpu_run(w, X, y, chain=chain, resident=True)
    assert np.array_equal(got, again)                # whichever workgroup comes first


@pytest.mark.parametrize("p,M,n", [(100, 84, 700), (100, 85, 588), (100, 85, 589),       # around the line to the staged kernel
                                   (101, 12, 1999), (101, 12, 2000),
                                   (100, 90, 577), (100, 86, 768), (127, 100, 769),      # shares of 148, 192 and 196 rows (48 at a time, eight to a chunk)
                                   (128, 400, 257),
                                   (112, 48, 2000), (112, 49, 2000), (100, 105, 559), (100, 105, 560),      # ... and around its other lines
                                   (97, 102, 700), (97, 103, 700), (99, 205, 599), (99, 205, 600), (128, 128, 600), (128, 129, 600)])
def test_shapes_against_the_oracle(p, M, n):
    w = _case(p, M * n, n, T=1)
    X, y = wl.dataset(w)
    got, _ = gpu_run(w, X, y, chain=3)
    assert rel_l2(got, oracle_run(w, X, y)) <= 1e-4


@pytest.mark.parametrize("p,M", [(99, 90), (99, 105), (128, 110)])
def test_a_pass_gives_the_same_bits_in_any_launch(p, M):
    """Five passes in launches of four and one, and one pass a launch; fixed partitions with cached matrices and without."""
    import torch
    import paper_2312_08728_amd as B
    w = _case(p, M * 601, 601, T=5)
    X, y = wl.dataset(w)
    a, _ = gpu_run(w, X, y, chain=3, reshuffle=1)
    b, _ = gpu_run(w, X, y, chain=3, reshuffle=1, cache_moments=True)
    assert np.array_equal(a, b)
    xd, yd, s = torch.from_numpy(X[:w.N0]).cuda(), torch.from_numpy(y[:w.N0]).cuda(), torch.cuda.Stream()
    got = []
    for chain_passes in (5, 1):
        ctx = B.Context(w.p, w.N0, w.n, w.alpha, 5, model=w.model, chain=3, reshuffle=1, n_buffers=1)
        ctx.set_passes(chain_passes)
        for _ in range(5 // chain_passes):
            ctx.run_device_buffer(xd, yd, w.N0, s)
        got.append(ctx.get_theta())
        ctx.close()
    assert np.array_equal(got[0], got[1])


def test_rows_of_a_subset():
    import torch
    import paper_2312_08728_amd as B
    w = _case(96, 90 * 600, 600, T=1)
    X, y = wl.dataset(w)
    rows = np.sort(np.random.default_rng(3).permutation(w.N0)[:86 * 600 + 7]).astype(np.int32)
    s, got = torch.cuda.Stream(), []
    for take in (False, True):                       # the listed rows, and the same rows as a buffer of their own
        Xs, ys = (X[:w.N0][rows], y[:w.N0][rows]) if take else (X[:w.N0], y[:w.N0])
        xd, yd = torch.from_numpy(np.ascontiguousarray(Xs)).cuda(), torch.from_numpy(np.ascontiguousarray(ys)).cuda()
        ctx = B.Context(w.p, w.N0, w.n, w.alpha, 1, model=w.model, chain=3)
        if not take:
            sub = torch.from_numpy(rows).cuda()
            ctx.set_row_subset(sub, len(rows))
        ctx.run_device_buffer(xd, yd, len(rows) if take else w.N0, s)
        got.append(ctx.get_theta())
        ctx.close()
    assert np.array_equal(got[0], got[1])
