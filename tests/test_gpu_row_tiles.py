"""The orders 5-7 stage on 16-element tiles on the GPU: from 72 tiles on
(K >= 1137) contexts run it instead of one element per workgroup.  Right-hand
side and one LSRK step against the FP64 oracle on both sides of that line, with
a ragged last tile, and batches that hold both kinds."""
import numpy as np
import pytest

import synth
from gpu_common import assert_parity, make_pair

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,N,precision,flux,bound",
                         [(5, 5, "fp32", "upwind", 2e-5), (6, 5, "fp32", "upwind", 2e-5),
                          (6, 5, "fp32", "central", 2e-5), (6, 6, "fp32", "upwind", 2e-5),
                          (6, 5, "bf16x3", "upwind", 1e-4), (6, 6, "bf16x3", "central", 1e-4),
                          (6, 7, "bf16x3", "upwind", 1e-4)])
def test_row_tiles_match_the_oracle(n, N, precision, flux, bound):
    print(f"case row tiles n={n} N={N} {precision} {flux}", flush=True)
    vx = synth.split_tet_vertices(synth.kuhn_cube_vertices(n))   # K = 6 n^3 + 3
    op, s = make_pair(n, N, synth.fourier_media, flux, precision, vertices=vx)
    q = synth.random_state(op.K, op.Np, seed=90 + N).astype(np.float32).astype(np.float64)
    got = s.rhs(torch.from_numpy(q).to("cuda:0", torch.float32)).cpu().numpy()
    assert_parity(got, op.rhs(q), bound, "rhs")
    ref, _ = op.step(q, np.zeros_like(q), 1e-3)
    s.set_state(q)
    s.step(0.0, 1e-3)
    assert_parity(s.get_state(), ref, bound, "one step")
    s.close()


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
def test_batch_of_both_kinds_equals_each_alone(precision):
    """Order 5, K = 162 and 384 (one element per workgroup) around 1,299
    (tiles): bit for bit as each context alone."""
    from paper_2008_09441_amd import B, Solver
    print(f"case batch of both kinds {precision}", flush=True)

    def make(n, seed, stream):
        s = Solver(5, precision=precision, device=0, stream=stream.cuda_stream)
        vx = synth.kuhn_cube_vertices(n)
        s.upload_mesh(synth.split_tet_vertices(vx) if n == 6 else vx)
        s.upload_media(synth.fourier_media)
        K, Np, _, _ = s.sizes()
        s.set_state(synth.random_state(K, Np, seed=seed))
        return s
    sizes, dt, st = (3, 6, 4), 1e-3, torch.cuda.Stream()
    alone = []
    for i, n in enumerate(sizes):
        s = make(n, 300 + i, st)
        B.dg_advance(s.ctx, dt, 3)
        alone.append(s.get_state())
        s.close()
    ctxs = [make(n, 300 + i, st) for i, n in enumerate(sizes)]
    b = B.dg_batch_create(0, 4)
    try:
        B.dg_batch_advance(b, st.cuda_stream, [s.ctx for s in ctxs], [dt] * 3, 3)
        for s, ref in zip(ctxs, alone):
            assert np.array_equal(s.get_state(), ref)
    finally:
        B.dg_batch_destroy(b)
        for s in ctxs:
            s.close()
