"""The step with a PML in every launch variant: streamed state, tile order, packed records and
speculative gathers leave the traces as they are, bit for bit, and a requested variant is the one
that runs.  Widths with one and with several lanes a node, 2D and 3D, ragged last batches."""
import numpy as np
import pytest

from synth import configs, pml

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N,steps", [(2, 45, 160), (3, 12, 140)])
@pytest.mark.parametrize("prec,widths", [(64, (1, 2, 8, 32)), (32, (1, 4, 16, 64))])
def test_every_variant(d, N, steps, prec, widths):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_04605_amd as mgrt
    p = configs.make("c1" if d == 2 else "c5", pml=True, N=N, L=0, n_src=11, n_steps=steps)
    p.pml = pml.pml_coefficients(p.mesh.centroids, 1.0, 1.5, 5.0)
    ctx = mgrt.context_for_problem(p)
    for b in widths:
        ref = None
        for v in range(16):
            y = ctx.forward_traces(p.src, p.rec[:, :1], p.wavelet, p.dt, steps, precision=prec, batch=b,
                                   launch=v + 1)
            assert ctx.last_timing()["variant"] == v
            ref = y if ref is None else ref
            assert np.array_equal(y, ref), (b, v)


def test_layer_changes_what_was_timed():
    """Adding and removing a layer times the variants and widths again: the choice for one step is
    none for the other."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_04605_amd as mgrt
    p = configs.make("c1", pml=True, N=256, L=0, n_src=16, n_steps=128)
    ctx = mgrt.context_for_problem(p)
    kw = dict(precision=32, one_step=True)
    args = (p.src, p.rec[:, :1], p.wavelet, p.dt, p.n_steps)
    tuned = []
    for layer in (True, True, False, True):
        ctx.upload_pml(*(p.pml if layer else (None, None)))
        ctx.forward_traces(*args, **kw)
        tuned.append(any(ctx.last_timing()["tune_us"]))
    assert tuned == [True, False, True, True]
