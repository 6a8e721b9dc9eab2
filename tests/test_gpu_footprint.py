"""dg_footprint against what a context holds (dg_memory), at every order and
precision: never less, and more by no more than the face-pattern table, which it
counts at its largest size (96 permutations of a face's nodes), so that a
scheduler refuses no request that fits."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7])
def test_footprint_is_what_the_context_holds(N, precision):
    from paper_2008_09441_amd import B, PRECISIONS, Solver
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case footprint N={N} {precision}", flush=True)
    s = Solver(N, precision=precision, device=0)
    s.upload_mesh(synth.kuhn_cube_vertices(3))
    s.upload_media(synth.homogeneous_media)
    s.set_sources([[0.3, 0.4, 0.6]], [[0.0, 1.0, 0.0]], 6.0, 0.2, 1.0)
    s.set_receivers(np.random.default_rng(1).random((5, 3)))
    B.dg_trace_reserve(s.ctx, 7)
    B.dg_state_zero(s.ctx)
    K, _, Nfp, _ = s.sizes()
    used, most = B.dg_memory(s.ctx), B.dg_footprint(N, PRECISIONS[precision], K, 1, 5, 7)
    s.close()
    print(f"{used} bytes held, {most} counted", flush=True)
    assert used <= most <= used + 96 * Nfp * 4
