"""Several leap-frog steps per launch for runs of several columns: one tile that holds the
mesh, regions of compact tiles, and strips of a lexicographic 2D grid.  Every node update is
the one-step launch's with its rounding, so the traces are equal bit for bit; step counts
that leave a remainder, columns that leave a ragged group, sources and receivers in many
tiles' halos."""
import numpy as np
import pytest

from oracle import Oracle
from synth import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mgrt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_04605_amd as m
    return m


def _both(ctx, p, rec, prec):
    args = (p.src, rec, p.wavelet, p.dt, p.n_steps)
    y1 = ctx.forward_traces(*args, precision=prec, one_step=True)
    assert ctx.last_timing()["steps_per_launch"] == 1
    return y1, ctx.forward_traces(*args, precision=prec), ctx.last_timing()


# one tile (2D up to 2,048 nodes, 3D up to 4,096), regions with one column a group (k = 12)
# and four or two, strips (k = 8, FP64 6) with 7 or 5 steps left over, 3D regions (k = 4)
@pytest.mark.parametrize("cfg,N,src,steps,prec,k", [
    ("c1", 24, 2, 257, 64, 64), ("c1", 44, 5, 320, 32, 64), ("c1", 45, 3, 300, 32, 12),
    ("c1", 45, 3, 301, 64, 12), ("c1", 96, 23, 300, 32, 8), ("c1", 150, 15, 263, 64, 8),
    ("c1", 300, 33, 303, 32, 8), ("c1", 300, 31, 263, 64, 6), ("c1", 301, 64, 258, 32, 8),
    ("c4", 12, 4, 300, 64, 64), ("c4", 16, 5, 257, 32, 4), ("c4", 24, 3, 300, 32, 4)])
def test_several_columns_equal_one_step(mgrt, cfg, N, src, steps, prec, k):
    p = configs.make(cfg, N=N, L=0, n_src=src, n_steps=steps)
    rec = np.stack([p.rec[:, 0], 0.3 * p.rec[:, 0] + 0.01], axis=1)
    ctx = mgrt.context_for_problem(p)
    y1, ym, t = _both(ctx, p, rec, prec)
    assert t["steps_per_launch"] == k and t["step_launches"] < p.n_steps
    assert np.array_equal(ym, y1)
    ref = Oracle.from_problem(p).forward(p.src[:2], rec[:2], p.wavelet, p.dt, p.n_steps)
    err = float(np.linalg.norm(ym[:2] - ref) / np.linalg.norm(ref))
    print(f"{cfg} N={N} {src} columns prec={prec}: {k} steps per launch, vs oracle {err:.2e}")
    assert err <= (1e-11 if prec == 64 else 1e-4)


def test_renumbered_grid_takes_regions(mgrt):
    """A 2D grid whose nodes come in random order is no lexicographic grid: regions of tiles
    cut by coordinates, whatever the stepping order."""
    p = configs.make("c1", N=300, L=0, n_src=32, n_steps=260)
    ms = p.mesh
    perm = np.random.default_rng(3).permutation(ms.coords.shape[0])
    inv = np.argsort(perm)
    ctx = mgrt.Context(0)
    ctx.upload_mesh(2, ms.coords[perm], inv[ms.elems], inv[ms.bfacets])
    ctx.upload_permittivity(p.eps)
    y1, ym, t = _both(ctx, p, p.rec, 32)
    assert t["steps_per_launch"] == 8 and np.array_equal(ym, y1)


def test_more_taps_than_a_tile_holds_take_one_step(mgrt):
    p = configs.make("c1", N=60, L=0, n_src=2, n_steps=260)
    rec = np.repeat(p.rec, 30, axis=1)               # 90 taps in one place
    ctx = mgrt.context_for_problem(p)
    y1, ym, t = _both(ctx, p, rec, 64)
    assert t["steps_per_launch"] == 1 and np.array_equal(ym, y1)


@pytest.mark.parametrize("N,src,prec", [(32, 5, 64), (64, 6, 32), (328, 16, 32)])
def test_jacobian_histories_equal_one_step(mgrt, N, src, prec):
    """Coarse-node histories written from regions and strips, against a requested batch width
    (one launch per step): the same values, so the same J bit for bit."""
    p = configs.make("c3", N=N, L=3, n_src=src, n_steps=700, n_samples=12)
    ctx = mgrt.context_for_problem(p)
    kw = dict(mode="mg", precision=prec)
    a = ctx.jacobian_coarse(p.src, p.rec, p.wavelet, p.dt, p.n_steps, p.sample_steps, **kw)
    t = ctx.last_timing()
    assert t["steps_per_launch"] > 1
    b = ctx.jacobian_coarse(p.src, p.rec, p.wavelet, p.dt, p.n_steps, p.sample_steps,
                            batch=t["batch"], **kw)
    assert ctx.last_timing()["steps_per_launch"] == 1
    assert np.array_equal(a, b)


@pytest.mark.parametrize("L,prec", [(1, 32), (1, 64), (2, 32)])
def test_jacobian_histories_in_neighbouring_rows(mgrt, L, prec):
    """Strips whose launches meet coarse nodes in several of a wave's rows at once."""
    p = configs.make("c3", N=512, L=L, n_src=16 if prec == 64 else 32, n_steps=270, n_samples=3)
    ctx = mgrt.context_for_problem(p)
    kw = dict(mode="mg", precision=prec)
    a = ctx.jacobian_coarse(p.src, p.rec, p.wavelet, p.dt, p.n_steps, p.sample_steps, **kw)
    t = ctx.last_timing()
    assert t["steps_per_launch"] == (8 if prec == 32 else 6)
    b = ctx.jacobian_coarse(p.src, p.rec, p.wavelet, p.dt, p.n_steps, p.sample_steps, batch=t["batch"], **kw)
    assert ctx.last_timing()["steps_per_launch"] == 1
    assert np.array_equal(a, b)


# regions with one, two and four columns a group, strips, one tile, 3D regions and 3D one-step
# launches; batches that leave a ragged one
@pytest.mark.parametrize("cfg,N,L,src,steps,prec,level", [
    ("c1", 24, 2, 2, 300, 64, "coarse"), ("c1", 45, 0, 3, 301, 64, "fine"), ("c1", 48, 2, 1, 300, 64, "coarse"),
    ("c1", 96, 3, 23, 300, 32, "coarse"), ("c1", 300, 2, 33, 263, 32, "fine"), ("c1", 300, 2, 9, 263, 64, "coarse"),
    ("c1", 400, 2, 64, 265, 32, "fine"), ("c1", 400, 2, 32, 263, 64, "coarse"),
    ("c4", 12, 1, 4, 300, 64, "coarse"), ("c4", 24, 1, 3, 270, 32, "coarse"), ("c4", 48, 0, 16, 260, 32, "fine")])
def test_gradient_with_all_velocities_kept(mgrt, cfg, N, L, src, steps, prec, level):
    """One segment (both sweeps several steps per launch) against checkpointed segments of one
    step per launch: equal fields, so the gradients differ by the order in which a node adds up
    its steps' and columns' products, steps * columns * 2^-53 <= 1e-12 of their magnitudes."""
    p = configs.make(cfg, N=N, L=L, n_src=src, n_steps=steps)
    rec = p.rec[:, :1]
    res = np.random.default_rng(5).standard_normal((src, 1, steps))
    ctx = mgrt.context_for_problem(p)
    args = (p.src, rec, p.wavelet, p.dt, steps, res, level)
    a = ctx.misfit_gradient(*args, precision=prec)
    t = ctx.last_timing()
    n = p.mesh.coords.shape[0]
    assert t["node_updates"] == 2 * n * steps * src
    # enough for states, checkpoints and a segment of about sqrt(2 * steps) steps, not for all
    slab = n * t["batch"] * (prec // 8)
    b = ctx.misfit_gradient(*args, precision=prec, batch=t["batch"] if src > 1 else 0, launch=4,
                            mem_budget_gb=(2 * np.sqrt(2 * steps) + 20) * slab / 2**30)
    tb = ctx.last_timing()
    assert tb["steps_per_launch"] == 1 and tb["node_updates"] == 3 * n * steps * src
    err = float(np.linalg.norm(a - b) / np.linalg.norm(b))
    print(f"{cfg} N={N} {src} columns prec={prec}: {t['steps_per_launch']} steps per launch, {err:.2e}")
    assert err <= 1e-12
