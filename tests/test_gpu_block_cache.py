"""Device blocks that wait between calls: reused by another context, bounded by a call's memory
budget, and given back on request and with a context."""
import numpy as np
import pytest

from synth import configs

pytestmark = pytest.mark.gpu

GB = 1 << 30


@pytest.fixture(scope="module")
def mgrt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_04605_amd as m
    return m


@pytest.fixture(scope="module")
def work():
    """A gradient whose velocities of all steps take 2 GB: 201^2 nodes, 32 columns, 400 steps."""
    p = configs.make("c1", N=200, L=2, n_src=32, n_steps=400)
    res = np.random.default_rng(11).standard_normal((32, 1, p.n_steps))
    return p, (p.src, p.rec[:, :1], p.wavelet, p.dt, p.n_steps, res, "fine")


def free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_release_gives_back(mgrt, work):
    p, args = work
    ctx = mgrt.context_for_problem(p)
    ctx.forward_traces(p.src, p.rec, p.wavelet, p.dt, 16, precision=32)
    ctx.release_cached()
    f0 = free()
    g = ctx.misfit_gradient(*args, precision=32)
    assert f0 - free() > 1.5 * GB                    # waiting
    ctx.release_cached()
    assert f0 - free() < GB // 4                     # operators and tables stay
    assert np.array_equal(ctx.misfit_gradient(*args, precision=32), g)


def test_two_contexts_share_blocks(mgrt, work):
    """Blocks are handed on with what the first context left in them."""
    p, args = work
    a, b = mgrt.context_for_problem(p), mgrt.context_for_problem(p)
    a.release_cached()
    g = a.misfit_gradient(*args, precision=32)
    f1 = free()
    h = b.misfit_gradient(*args, precision=32)
    assert f1 - free() < GB // 4
    assert np.array_equal(g, h)
    a.close()
    assert free() - f1 > 1.5 * GB                    # b is still there
    assert np.array_equal(b.misfit_gradient(*args, precision=32), g)


def test_budget_bounds_what_waits(mgrt, work):
    p, args = work
    ctx = mgrt.context_for_problem(p)
    ctx.forward_traces(p.src, p.rec, p.wavelet, p.dt, 16, precision=32)
    ctx.release_cached()
    f0 = free()
    ctx.misfit_gradient(*args, precision=32)
    assert f0 - free() > 1.5 * GB
    ctx.misfit_gradient(*args, precision=32, mem_budget_gb=0.5)
    assert f0 - free() < 0.5 * GB + GB // 4


def test_two_threads_share_blocks(mgrt, work):
    """Two contexts on two threads give and take blocks while the other one runs, captures and
    replays: the same results as one after the other."""
    import threading
    p, args = work
    q = configs.make("c1", N=260, L=0, n_src=32, n_steps=600)
    a, b = mgrt.context_for_problem(p), mgrt.context_for_problem(q)

    def gradients():
        return [a.misfit_gradient(*args, precision=32) for _ in range(8)]

    def forwards():
        return [b.forward_traces(q.src, q.rec, q.wavelet, q.dt, q.n_steps, precision=prec)
                for prec in (32, 64) * 5]

    ref = gradients(), forwards()
    got = [None, None]

    def run(i, fn):
        got[i] = fn()
    threads = [threading.Thread(target=run, args=(i, fn)) for i, fn in enumerate((gradients, forwards))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for x, y in zip(ref, got):
        assert y is not None and all(np.array_equal(u, v) for u, v in zip(x, y))
