"""The moment matrices of up to 47 features formed straight from gathered rows (64 mini-batches a pass or more): tile and row-share edges,
entries of the partition worked out on the way, one and two workgroups per mini-batch.  fp32 sums, as in the other tests of this form: 1e-4."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import gpu_run, oracle_run, rel_l2

pytestmark = pytest.mark.gpu


def _case(p, N0, n, T, R=1):
    return wl.CONFIGS["cfg2"].scaled(name="case", N=2 * N0 - 5, p=p, N0=N0, n=n, T=T, R=R, alpha=0.1 / (p + 10), x_cov="identity")


@pytest.mark.parametrize("chain", [3, 5])            # the chain's layout, and dense for the products
@pytest.mark.parametrize("n", [101, 773])            # one workgroup per mini-batch, and two
@pytest.mark.parametrize("p", [1, 2, 15, 16, 17, 31, 32, 46, 47])
def test_tile_edges_against_the_oracle(p, n, chain):
    """65 mini-batches (shares of 28 and 100 rows, the last ones short) and one of 3 rows; a second buffer of 5 rows less."""
    w = _case(p, 65 * n + 3, n, 2)
    X, y = wl.dataset(w)
    got, st = gpu_run(w, X, y, chain=chain)
    assert st.chain == chain and rel_l2(got, oracle_run(w, X, y)) <= 1e-4
    again, _ = gpu_run(w, X, y, chain=chain, resident=True)
    assert np.array_equal(got, again)                # whichever workgroup comes first


@pytest.mark.parametrize("p,N0,n", [(20, 64 * 40, 40),        # the fewest mini-batches; shares of 12 rows
                                    (20, 63 * 40, 40),        # one fewer: the staged kernel
                                    (7, 511 * 15, 15),        # shares of 4 rows
                                    (20, 64 * 10, 10),        # and a wavefront without any
                                    (7, 160 * 768, 768),      # two workgroups per mini-batch (96 rows a share)
                                    (7, 161 * 768, 768),      # one
                                    (7, 161 * 1024, 1024),    # two
                                    (3, 512 * 1024, 1024),    # one: so many mini-batches fill the device
                                    (30, 64 * 2100, 2100)])   # shares of 264 rows: several times 64 entries of the partition
def test_shapes_against_the_oracle(p, N0, n):
    w = _case(p, N0, n, 2)
    X, y = wl.dataset(w)
    got, _ = gpu_run(w, X, y, chain=3)
    assert rel_l2(got, oracle_run(w, X, y)) <= 1e-4


def test_fixed_partitions_cached_and_not_are_the_same_bits():
    w = _case(12, 70 * 33, 33, 3, R=2)
    X, y = wl.dataset(w)
    a, _ = gpu_run(w, X, y, chain=3, reshuffle=1)
    b, _ = gpu_run(w, X, y, chain=3, reshuffle=1, cache_moments=True)
    assert np.array_equal(a, b)
