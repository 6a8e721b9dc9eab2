"""Orders 2-4 on both sides of the line between one element per workgroup and
16-element tiles (24, 48 and 64 tiles): right-hand side and one LSRK step
against the FP64 oracle, with a ragged last tile where the mesh is split, and a
batch of both kinds bit for bit as each context alone."""
import numpy as np
import pytest

import synth
from gpu_common import assert_parity, make_pair

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOUND = {"fp64": 1e-12, "fp32": 2e-5, "bf16x3": 1e-4}


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# tiles: 11 and 25 (order 2), 47 and 82 (orders 3 and 4)
@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("n,N", [(3, 2), (4, 2), (5, 3), (6, 3), (5, 4), (6, 4)])
def test_both_sides_match_the_oracle(n, N, precision):
    print(f"case small mesh n={n} N={N} {precision}", flush=True)
    vx = synth.split_tet_vertices(synth.kuhn_cube_vertices(n)) if n != 5 else None
    op, s = make_pair(n, N, synth.fourier_media, "upwind", precision, vertices=vx)
    q = synth.random_state(op.K, op.Np, seed=110 + N)
    dtype = torch.float64 if precision == "fp64" else torch.float32
    if precision != "fp64":
        q = q.astype(np.float32).astype(np.float64)
    got = s.rhs(torch.from_numpy(q).to("cuda:0", dtype)).cpu().numpy()
    assert_parity(got, op.rhs(q), BOUND[precision], "rhs")
    ref, _ = op.step(q, np.zeros_like(q), 1e-3)
    s.set_state(q)
    s.step(0.0, 1e-3)
    assert_parity(s.get_state(), ref, BOUND[precision], "one step")
    s.close()


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
def test_batch_of_both_kinds_equals_each_alone(precision):
    from paper_2008_09441_amd import B, Solver
    print(f"case batch of both kinds, order 3 {precision}", flush=True)

    def make(n, seed, stream):
        s = Solver(3, precision=precision, device=0, stream=stream.cuda_stream)
        s.upload_mesh(synth.kuhn_cube_vertices(n))
        s.upload_media(synth.fourier_media)
        K, Np, _, _ = s.sizes()
        s.set_state(synth.random_state(K, Np, seed=seed))
        return s
    sizes, dt, st = (6, 3, 7, 4), 1e-3, torch.cuda.Stream()
    alone = []
    for i, n in enumerate(sizes):
        s = make(n, 400 + i, st)
        B.dg_advance(s.ctx, dt, 3)
        alone.append(s.get_state())
        s.close()
    ctxs = [make(n, 400 + i, st) for i, n in enumerate(sizes)]
    try:
        B.dg_batch_advance_noalloc(st.cuda_stream, [s.ctx for s in ctxs], [dt] * 4, 3)
        for s, ref in zip(ctxs, alone):
            assert np.array_equal(s.get_state(), ref)
    finally:
        for s in ctxs:
            s.close()
