"""The stage kernel of a context that may be batched: at orders 2-4 FP32 and
BF16x3 contexts run 16-element tiles at every size, since a batch fills the chip
with the tiles of all of its contexts, however few each of them has; at orders
5-7 a context runs tiles from the size on at which a batch that also holds smaller
contexts (one element per workgroup, in a launch of their own) does not pay for
it.  Times against the same kernels of this library, by medians of five."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N", [1, 2, 3, 4])
def test_tiled_contexts_hold_the_same_arrays_at_every_size(N):
    """BF16x3 at orders 1-4: bytes per 16 elements do not depend on the size (a
    context that ran one element per workgroup would hold a second copy of its
    material)."""
    from paper_2008_09441_amd import B

    def per_tile(K):
        return (B.dg_footprint(N, B.DG_FP32_BF16X3, K + 16) - B.dg_footprint(N, B.DG_FP32_BF16X3, K))
    assert per_tile(160) == per_tile(16000)


def _context(n, N, precision, stream):
    from paper_2008_09441_amd import Solver
    s = Solver(N, precision=precision, device=0, stream=stream.cuda_stream)
    s.upload_mesh(synth.kuhn_cube_vertices(n))
    s.upload_media(synth.homogeneous_media)
    K, Np, _, _ = s.sizes()
    s.set_state(synth.random_state(K, Np, seed=n))
    return s


def _time(ns, N, precision, steps=10):
    """us of a stage of the batch of contexts of 6 n^3 elements, n in ns."""
    from paper_2008_09441_amd import B
    st = torch.cuda.Stream()
    cs = [_context(n, N, precision, st) for n in ns]
    b = B.dg_batch_create(0, len(cs))
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    out = []
    try:
        with torch.cuda.stream(st):
            for _ in range(6):
                ev[0].record()
                B.dg_batch_advance(b, st.cuda_stream, [c.ctx for c in cs], [1e-6] * len(cs), steps)
                ev[1].record()
                torch.cuda.synchronize()
                out.append(ev[0].elapsed_time(ev[1]) * 1e3 / (5 * steps))
    finally:
        B.dg_batch_destroy(b)
        for c in cs:
            c.close()
    return float(np.median(out[1:]))


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("N,small,large", [(2, 3, 6), (3, 5, 10), (4, 5, 10)])
def test_eight_small_contexts_cost_what_one_large_one_does(N, small, large, precision):
    """Eight contexts, each an eighth of the elements of one context: at most 1.6
    times its time (one element per workgroup would take 1.9 to 3.7 times)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case eight small contexts N={N} {precision}", flush=True)
    one, eight = _time([large], N, precision), _time([small] * 8, N, precision)
    print(f"one {one:.1f} us, eight {eight:.1f} us a stage", flush=True)
    assert eight <= 1.6 * one


@pytest.mark.gpu
@pytest.mark.parametrize("N", [5, 6])
def test_a_batch_is_faster_than_its_contexts_in_turn(N):
    """BF16x3, 1,296 and 384 elements: one launch a stage for both (two launches
    would take as long as the contexts in turn)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case batch against its contexts N={N}", flush=True)
    a, c, both = _time([6], N, "bf16x3"), _time([4], N, "bf16x3"), _time([6, 4], N, "bf16x3")
    print(f"{a:.1f} + {c:.1f} us alone, {both:.1f} us together a stage", flush=True)
    assert both <= 0.95 * (a + c)
