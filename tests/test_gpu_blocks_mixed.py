"""Several steps per launch on ONE context that is used at both precisions and with changing
numbers of sources, as an interactive session does.  Most shapes are ones where FP32 columns in
groups of four and FP64 columns in pairs ask for the same number of tiles and steps: their
tables differ all the same."""
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


@pytest.mark.parametrize("N,calls", [
    (64, ((32, 64), (64, 64), (32, 64))), (128, ((32, 16), (64, 8), (32, 16))),
    (96, ((64, 32), (32, 64), (64, 32))), (300, ((32, 33), (64, 31), (32, 12)))])
def test_forward_at_both_precisions(mgrt, N, calls):
    p = configs.make("c1", N=N, L=0, n_src=64, n_steps=263)
    ctx = mgrt.context_for_problem(p)
    for prec, src in calls:
        args = (p.src[:src], p.rec[:src], p.wavelet, p.dt, p.n_steps)
        y = ctx.forward_traces(*args, precision=prec)
        t = ctx.last_timing()
        assert t["steps_per_launch"] > 1
        y1 = ctx.forward_traces(*args, precision=prec, one_step=True)
        assert ctx.last_timing()["steps_per_launch"] == 1
        print(f"N={N} fp{prec} {src} sources: {t['steps_per_launch']} steps per launch", flush=True)
        assert np.array_equal(y, y1), (prec, src)


@pytest.mark.parametrize("N,calls", [(128, ((32, 16), (64, 8), (32, 16))), (96, ((64, 32), (32, 64), (64, 32)))])
def test_gradient_at_both_precisions(mgrt, N, calls):
    """The mixed context against a fresh one per call: the same launches, so equal bit for bit."""
    p = configs.make("c1", N=N, L=2, n_src=64, n_steps=261)
    res = np.random.default_rng(7).standard_normal((64, 1, p.n_steps))
    ctx = mgrt.context_for_problem(p)
    for prec, src in calls:
        args = (p.src[:src], p.rec[:src, :1], p.wavelet, p.dt, p.n_steps, res[:src], "fine")
        g = ctx.misfit_gradient(*args, precision=prec)
        assert ctx.last_timing()["steps_per_launch"] > 1
        ref = mgrt.context_for_problem(p).misfit_gradient(*args, precision=prec)
        print(f"N={N} fp{prec} {src} sources", flush=True)
        assert np.array_equal(g, ref), (prec, src)
