"""The step with a PML in one launch (the layer's state in its first workgroups) at every batch
width, in 2D and 3D, with columns that leave a ragged last batch, against the mixed-form oracle.
Tolerances as for all forward runs: FP64 1e-11, FP32 1e-4."""
import numpy as np
import pytest

from oracle import Oracle
from synth import configs, pml

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N,steps", [(2, 45, 400), (3, 12, 120)])
@pytest.mark.parametrize("prec,widths", [(64, (1, 2, 4, 8, 16, 32, 64, 128)), (32, (1, 4, 8, 16, 32, 64, 128))])
def test_every_width(d, N, steps, prec, widths):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_04605_amd as mgrt
    p = configs.make("c1" if d == 2 else "c5", pml=True, N=N, L=0, n_src=11, n_steps=steps)
    # a layer that these meshes resolve (dt zeta about 0.35)
    p.pml = pml.pml_coefficients(p.mesh.centroids, 1.0, 1.5, 5.0)
    rec = p.rec[:, :1]
    ref = Oracle.from_problem(p).forward(p.src, rec, p.wavelet, p.dt, steps)
    ctx = mgrt.context_for_problem(p)
    for b in widths:
        y = ctx.forward_traces(p.src, rec, p.wavelet, p.dt, steps, precision=prec, batch=b)
        err = float(np.linalg.norm(y - ref) / np.linalg.norm(ref))
        print(f"{d}D N={N} fp{prec} batch {b}: {err:.2e}")
        assert err <= (1e-11 if prec == 64 else 1e-4), b
