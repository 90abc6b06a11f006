"""Lagged sums of the Jacobian where later impulse-response samples are not finite (a run above
the stability bound): a sum uses the samples up to its own step only, so the early rows are
those of a call that asks for no later one."""
import numpy as np
import pytest

from synth import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,steps,late", [(32, 120, 119), (64, 700, 650)])
def test_early_sums_do_not_see_later_samples(prec, steps, late):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_04605_amd as mgrt
    from paper_1707_04605_amd import native
    p = configs.make("c3", N=32, L=2, n_src=3, n_steps=steps, n_samples=4)
    ctx = mgrt.context_for_problem(p)
    dt = 2.0 * ctx.stability_bound()               # every step multiplies the field by about 14
    plain = ctx._opts
    ctx._opts = lambda precision, variant, batch, timing, flags, *more: plain(
        precision, variant, batch, timing, flags | native.F_SKIP_STABILITY, *more)

    def rows(samples):
        out = torch.empty(3 * len(samples), ctx.n_coarse, dtype=torch.float64, device="cuda")
        ctx.jacobian_coarse(p.src, p.rec[:, :1], p.wavelet, dt, steps, np.array(samples), precision=prec,
                            pairing="direct", out=out)
        return out.reshape(3, len(samples), -1).cpu().numpy()

    early, all_ = rows([3, 9]), rows([3, 9, late])
    assert np.isfinite(early).all() and (early != 0).any()
    assert not np.isfinite(all_[:, 2]).all()       # the late samples do overflow
    assert np.array_equal(all_[:, :2], early)
