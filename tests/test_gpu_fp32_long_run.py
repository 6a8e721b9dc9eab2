"""FP32 over many steps: the stage on three bf16 parts per operand (orders 3-6)
stays as close to FP64 as FP32 products do, which the forward run of the adjoint
keeps at every order.  A rounding that always goes one way would not show in one
right-hand side, but adds up over a run.  Bound: 1.06 times the error of the FP32
products; over media, fluxes and initial states the ratio of two FP32 runs that
both round to nearest scatters by 0.03 at most."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _state(x):
    """Three smooth waves in each field at the nodes x [K, Np, 3]."""
    rng = np.random.default_rng(5)
    q = np.zeros((9,) + x.shape[:-1])
    for f in range(9):
        for _ in range(3):
            k, ph = rng.integers(-2, 3, size=3), rng.uniform(0.0, 6.0)
            q[f] += 0.3 * np.sin(2.0 * np.pi * (x @ k) + ph)
    return q


@pytest.mark.parametrize("N", [3, 4, 5, 6])
def test_three_part_products_drift_no_more_than_fp32_products(N):
    from paper_2008_09441_amd import B, Solver
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case FP32 long run N={N}", flush=True)
    n, steps, every = 8, 800, 10
    dt = 0.5 / n / np.sqrt(2.0) / (4.0 * (N + 1) ** 2)
    end = {}
    for name, precision in (("fp64", "fp64"), ("parts", "fp32"), ("products", "fp32")):
        s = Solver(N, precision=precision, device=0)
        s.upload_mesh(synth.kuhn_cube_vertices(n))
        s.upload_media(synth.fourier_media)
        s.set_receivers([[0.3, 0.4, 0.6]])
        s.set_state(_state(s.node_coords()).astype(np.float32).astype(s.dtype))
        if name == "products":
            B.dg_adjoint_forward(s.ctx, 0.0, dt, steps, every, np.empty((steps, 1, 3), s.dtype))
        else:
            s.run(0.0, dt, steps)
        end[name] = s.get_state().astype(np.float64)
        s.close()
    err = {k: np.linalg.norm(end[k] - end["fp64"]) / np.linalg.norm(end["fp64"])
           for k in ("parts", "products")}
    print(f"error after {steps} steps: {err['parts']:.3e} (FP32 products {err['products']:.3e})",
          flush=True)
    assert err["parts"] <= 1.06 * err["products"]
