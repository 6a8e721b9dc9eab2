"""The generic adjoint's per-element kernels on both sides of the order at which
they give a thread three of the nine components of a row instead of all nine
(orders 1-3, order 4 on): gradients in the weights and the impedances against
the oracle's discrete adjoint, FP64, with checkpoint intervals of unequal length.
Tolerance: 1e-10, the bound of the FP64 gradients at every order."""
import numpy as np
import pytest

from oracle import adjoint as oadj
import test_gpu_adjoint as base

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,flux", [(1, "upwind"), (1, "central"), (3, "central"), (4, "upwind")])
def test_gradient_matches_the_oracle_on_both_sides_of_the_split(N, flux):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case adjoint split N={N} flux={flux}", flush=True)
    op, s, m, zp, zs, q0 = base._setup(flux, "fp64", n=2, N=N)
    z = np.stack([zp, zs])
    dt, nsteps, every = 0.005, 5, 3
    d = np.random.default_rng(31).standard_normal((nsteps, len(base.RECS), 3)) * 0.05
    tr_ref = oadj.forward_trace(op, m, q0, 0.0, dt, nsteps, base.SRC, base.RECS, z)
    g_ref, gz_ref = oadj.gradient(op, m, q0, 0.0, dt, nsteps, base.SRC, base.RECS, tr_ref - d,
                                  z=z, with_z=True)
    _, g, gz = base._gpu_grad_z(s, m, zp, zs, q0, dt, nsteps, every, d)
    assert np.linalg.norm(g - g_ref) <= 1e-10 * np.linalg.norm(g_ref)
    assert np.linalg.norm(gz - gz_ref) <= 1e-10 * np.linalg.norm(gz_ref)
