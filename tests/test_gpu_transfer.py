"""theta through pinned memory and back: estimates of one part, of exactly one area, of several, with a ragged last part."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,C", [(8, 2), (512, 512), (520, 513), (1032, 2047)])
def test_softmax_estimates_come_back_bit_for_bit(p, C):
    import paper_2312_08728_amd as B
    ctx = B.Context(p, 64, 64, 0.1, 1, model=B.BMGD_SOFTMAX, n_classes=C)
    try:
        assert not ctx.get_theta().any()
        w = np.random.default_rng(p).standard_normal((p, C)).astype(np.float32)
        ctx.set_theta(w)
        assert np.array_equal(ctx.get_theta(), w)
        ctx.swa_update()
        avg, count = ctx.get_swa()
        assert count == 1 and np.array_equal(avg, w)
    finally:
        ctx.close()


@pytest.mark.parametrize("p,model", [(1, 0), (37, 1), (4096, 0)])
def test_glm_estimates_come_back_bit_for_bit(p, model):
    import paper_2312_08728_amd as B
    ctx = B.Context(p, 64, 64, 0.1, 1, model=model)
    try:
        w = np.random.default_rng(p).standard_normal(p).astype(np.float32)
        ctx.set_theta(w)
        assert np.array_equal(ctx.get_theta(), w)
    finally:
        ctx.close()
