"""The 16-element tile kernels at the sizes that run them (which kernel a context
runs is a matter of its order, precision and number of tiles): central and upwind
flux against the FP64 oracle, batches of tiles and of both kinds with sources,
receivers and odd step counts against each context alone, and the FP32 adjoint at
an order and size whose plain runs take tiles.  Bounds as elsewhere: FP64 1e-12,
FP32 2e-5, BF16x3 1e-4; batches bit for bit; FP32 gradients 1e-5."""
import numpy as np
import pytest

import synth
import test_gpu_adjoint_tiled as adj
from gpu_common import assert_parity, make_pair
from test_gpu_serving import _ctx

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOUND = {"fp64": 1e-12, "fp32": 2e-5, "bf16x3": 1e-4}


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# with a ragged last tile (K = 6 n^3 + 3).  FP64 takes tiles from 24, 48 and 64
# tiles on at orders 2-4, the others at every size; orders 5-7 from 96 (FP32,
# order 7) and 128 (orders 5 and 6 BF16x3) on
@pytest.mark.parametrize("n,N,precision,flux", [
    (3, 1, "fp64", "central"), (5, 2, "fp64", "central"), (6, 3, "fp64", "central"),
    (6, 4, "fp64", "central"), (3, 1, "fp32", "central"), (3, 2, "fp32", "central"),
    (3, 3, "fp32", "central"), (4, 4, "fp32", "central"), (3, 1, "bf16x3", "central"),
    (3, 2, "bf16x3", "central"), (4, 3, "bf16x3", "central"), (3, 4, "bf16x3", "central"),
    (7, 5, "fp32", "upwind"), (7, 5, "fp32", "central"), (7, 6, "fp32", "upwind"),
    (7, 6, "fp32", "central"), (7, 5, "bf16x3", "upwind"), (8, 6, "bf16x3", "central"),
    (7, 7, "bf16x3", "upwind"), (7, 7, "bf16x3", "central")])
def test_tiles_match_the_oracle(n, N, precision, flux):
    print(f"case tiles n={n} N={N} {precision} {flux}", flush=True)
    vx = synth.split_tet_vertices(synth.kuhn_cube_vertices(n))
    op, s = make_pair(n, N, synth.fourier_media, flux, precision, vertices=vx)
    q = synth.random_state(op.K, op.Np, seed=130 + N)
    dtype = torch.float64 if precision == "fp64" else torch.float32
    if precision != "fp64":
        q = q.astype(np.float32).astype(np.float64)
    got = s.rhs(torch.from_numpy(q).to("cuda:0", dtype)).cpu().numpy()
    assert_parity(got, op.rhs(q), BOUND[precision], "rhs")
    ref, _ = op.step(q, np.zeros_like(q), 2e-4)
    s.set_state(q)
    s.step(0.0, 2e-4)
    assert_parity(s.get_state(), ref, BOUND[precision], "one step")
    s.close()


# sizes around the lines above: at orders 2-4 tiles only, at orders 5-7 both kinds
@pytest.mark.parametrize("N,precision,sizes", [
    (2, "fp32", (2, 3, 6)), (2, "bf16x3", (2, 6, 3)), (3, "fp32", (6, 2, 3)),
    (4, "fp32", (2, 6, 3)), (4, "bf16x3", (3, 2, 6)), (5, "fp32", (2, 7, 3)),
    (5, "bf16x3", (7, 2, 3)), (6, "fp32", (2, 3, 7)), (6, "bf16x3", (2, 8)),
    (7, "bf16x3", (2, 7))])
def test_batches_of_tiles_equal_each_context_alone(N, precision, sizes):
    from paper_2008_09441_amd import B
    print(f"case batch of tiles N={N} {precision} {sizes}", flush=True)
    steps = (3, 2)
    dts = [0.5 / n / np.sqrt(2.0) / (4.0 * (N + 1) ** 2) for n in sizes]

    def result(s):
        tr = np.empty((sum(steps), 4, 3), dtype=s.dtype)
        B.dg_trace_copy(s.ctx, tr, sum(steps))
        return tr, s.get_state(), B.dg_time_get(s.ctx)
    alone = []
    for i, n in enumerate(sizes):
        s = _ctx(n, N, precision, torch.cuda.Stream(), 500 + i, sum(steps))
        s.set_state(0.1 * synth.random_state(*s.sizes()[:2], seed=i))
        for k in steps:
            B.dg_advance(s.ctx, dts[i], k)
        alone.append(result(s))
        s.close()
    st = torch.cuda.Stream()
    ctxs = [_ctx(n, N, precision, st, 500 + i, sum(steps)) for i, n in enumerate(sizes)]
    b = B.dg_batch_create(0, len(sizes))
    try:
        for i, s in enumerate(ctxs):
            s.set_state(0.1 * synth.random_state(*s.sizes()[:2], seed=i))
        for k in steps:
            B.dg_batch_advance(b, st.cuda_stream, [s.ctx for s in ctxs], dts, k)
        for s, (tr, q, clock) in zip(ctxs, alone):
            got = result(s)
            assert np.abs(tr).max() > 0
            assert np.array_equal(got[0], tr) and np.array_equal(got[1], q) and got[2] == clock
    finally:
        B.dg_batch_destroy(b)
        for s in ctxs:
            s.close()


@pytest.mark.parametrize("flux", ["upwind", "central"])
def test_fp32_adjoint_of_order_5_where_plain_runs_take_tiles(flux):
    """2,058 elements: the forward run and the replay of the adjoint stay on one
    element per workgroup."""
    print(f"case FP32 adjoint N=5 on 2,058 elements {flux}", flush=True)
    n, N = 7, 5
    vx = synth.kuhn_cube_vertices(n)
    s64, m, zp = adj._solver(n, N, flux, "fp64", vx)
    s32, _, _ = adj._solver(n, N, flux, "fp32", vx)
    q0 = synth.random_state(*s64.sizes()[:2], seed=29) * 0.1
    dt, nsteps, every = 3e-4, 4, 3
    d = np.random.default_rng(27).standard_normal((nsteps, len(adj.RECS), 3)) * 0.05
    _, [(g64, z64)] = adj._grads(s64, m, zp, q0, dt, nsteps, every, d)
    _, [(g32, z32)] = adj._grads(s32, m, zp, q0, dt, nsteps, every, d)
    s64.close()
    s32.close()
    eg = adj._rel(g32, g64)
    print("gradient m per field:", np.array2string(eg, precision=2), flush=True)
    assert np.isfinite(g32).all() and eg.max() <= 1e-5
    if flux == "upwind":
        ez = adj._rel(z32, z64)
        print("gradient z per field:", np.array2string(ez, precision=2), flush=True)
        assert ez.max() <= 1e-5
    else:
        assert not z32.any()
