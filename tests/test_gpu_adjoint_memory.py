"""Device memory of an adjoint run against what include/dg.h states: checkpoints,
stage inputs (and, on the tiled FP32 kernels, R y and the face jumps of every stage
input, of two intervals), five state vectors, face-node arrays and gradients.  The
tables and fragments beside them are smaller than one state vector here."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,precision", [(4, "fp32"), (3, "fp64"), (5, "fp32")])
def test_adjoint_memory_is_what_the_header_states(N, precision):
    from paper_2008_09441_amd import B, Solver
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case adjoint memory N={N} {precision}", flush=True)
    s = Solver(N, precision=precision, device=0)
    s.upload_mesh(synth.kuhn_cube_vertices(5))
    s.upload_media(synth.homogeneous_media)
    s.set_receivers([[0.3, 0.4, 0.6]])
    B.dg_state_zero(s.ctx)
    K, Np, Nfp, Nq = s.sizes()
    before, steps, every = B.dg_memory(s.ctx), 5, 2
    B.dg_adjoint_forward(s.ctx, 0.0, 1e-4, steps, every, np.empty((steps, 1, 3), s.dtype))
    held = B.dg_memory(s.ctx) - before
    s.close()
    e = 8 if precision == "fp64" else 4
    tiled = precision == "fp32" and N <= 4
    face = K * 4 * Nfp * e
    state = 9 * K * Np * e
    stated = (3 + (20 if tiled else 5) * every + 5) * state       # checkpoints, inputs, vectors
    stated += (9 if tiled else 18) * face + 8 * (3 * K * Nq + 2 * K * Np)
    stated += (8 + 8 * 10 * every if tiled else 4) * face         # jumps, impedance terms
    print(f"{held} bytes held, {stated} stated, {state} a state vector", flush=True)
    assert stated <= held < stated + state
