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


@pytest.mark.parametrize("p,C,model", [(37, 1, 0), (64, 20, 2), (520, 513, 2)])
def test_a_failed_run_leaves_the_output_alone(p, C, model):
    """A run that failed (a row subset with an index outside its buffer) is reported before anything is written to the caller's
    array, also where an estimate comes back in several parts."""
    import torch
    import paper_2312_08728_amd as B
    rows = 64
    bf16 = model == B.BMGD_SOFTMAX
    x = torch.randn((rows, p), device="cuda", generator=torch.Generator(device="cuda").manual_seed(p))
    x = x.bfloat16() if bf16 else x
    y = torch.zeros(rows, dtype=torch.int32 if bf16 else torch.float32, device="cuda")
    bad = torch.arange(rows, dtype=torch.int32, device="cuda")
    bad[3] = rows
    ctx = B.Context(p, rows, 32, 0.01, 1, model=model, n_classes=C)
    try:
        for fetch in (lambda out: B.bmgd_get_theta(ctx.h, out, out.size), lambda out: B.bmgd_get_swa(ctx.h, out, out.size)[0]):
            ctx.set_row_subset(bad, rows)
            ctx.run_device_buffer(x, y, rows, None)
            ctx.swa_update()
            out = np.full(p * C, 7.0, dtype=np.float32)
            assert fetch(out) == B.BMGD_EINVAL
            assert (out == 7.0).all()
            ctx.set_theta(np.zeros(p * C, dtype=np.float32))
    finally:
        ctx.close()
