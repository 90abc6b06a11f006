"""When the tables of several-step launches are made and what they hold: one column on more than
65,536 nodes takes one step per launch until its runs repay them, with the same values before and
after; sources and receivers that move from call to call find their tiles."""
import numpy as np
import pytest

from synth import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mgrt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_04605_amd as m
    return m


@pytest.mark.parametrize("prec", [32, 64])
def test_short_one_column_runs_wait(mgrt, prec):
    p = configs.make("c1", N=300, L=0, n_src=1, n_steps=30)
    ctx = mgrt.context_for_problem(p)
    args = (p.src, p.rec, p.wavelet, p.dt, p.n_steps)
    ref = ctx.forward_traces(*args, precision=prec, one_step=True)
    k = []
    for _ in range(4):
        y = ctx.forward_traces(*args, precision=prec)
        k.append(ctx.last_timing()["steps_per_launch"])
        assert np.array_equal(y, ref)
    assert k == [1, 1, 12, 12]                       # 90 steps asked for at the third call


# one tile, regions of one and of four columns in 2D, regions in 3D
@pytest.mark.parametrize("cfg,N,src", [("c1", 30, 3), ("c1", 100, 4), ("c1", 140, 20), ("c4", 20, 3)])
def test_points_that_move(mgrt, cfg, N, src):
    p = configs.make(cfg, N=N, L=0, n_src=src, n_steps=260)
    ctx = mgrt.context_for_problem(p)
    rng = np.random.default_rng(N)
    for _ in range(4):
        a = rng.uniform(-1.4, 1.4, size=p.src.shape)
        r = rng.uniform(-1.5, 1.5, size=p.rec[:, :1].shape)
        args = (a, r, p.wavelet, p.dt, p.n_steps)
        y = ctx.forward_traces(*args, precision=32)
        assert ctx.last_timing()["steps_per_launch"] > 1
        assert np.array_equal(y, ctx.forward_traces(*args, precision=32, one_step=True))
