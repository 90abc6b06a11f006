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


def test_more_loads_than_a_tile_holds(mgrt):
    """Residuals of 30 receivers in one place: both sweeps take one launch per step, also where
    the forward sweep alone would not have to, with the values of a requested batch width."""
    p = configs.make("c1", N=60, L=0, n_src=4, n_steps=260)
    rec = np.repeat(p.rec[:, :1], 30, axis=1)
    res = np.random.default_rng(4).standard_normal((4, 30, p.n_steps))
    ctx = mgrt.context_for_problem(p)
    args = (p.src, rec, p.wavelet, p.dt, p.n_steps, res, "fine")
    a = ctx.misfit_gradient(*args, precision=64)
    t = ctx.last_timing()
    assert t["steps_per_launch"] == 1
    b = ctx.misfit_gradient(*args, precision=64, batch=t["batch"])
    # the same steps: equal but for the order in which a node adds up its columns
    assert float(np.linalg.norm(a - b) / np.linalg.norm(b)) <= 1e-12
