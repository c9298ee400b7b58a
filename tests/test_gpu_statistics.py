"""Bucket scope: the statistics of the last pass, kept in two sets by turns, against a context that clears one set before
every pass; passes over all nodes and single nodes, fits, and a captured pass replayed between them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2505_14371_amd import qoda  # noqa: E402


def test_two_sets_equal_one():
    if not torch.cuda.is_available():
        pytest.fail("a GPU test was selected but no GPU is visible")
    import gpu_harness

    sizes, K, S = [5000, 1, 0, 3 * 16384 + 7, 300], 3, 8
    two, one = [gpu_harness.GpuModel(sizes, [0, 1, 0, 1, 1], [S, S], K, seed=6, norm_scope=qoda.SCOPE_BUCKET) for _ in range(2)]
    one.ctx.profile_enable(["k_zero_u32"])
    graph = None
    rng = np.random.default_rng(1)
    t = 0

    def same():
        for which in (qoda.BUF_HIST, qoda.BUF_SUMSQ, qoda.BUF_DELTA, qoda.BUF_POOLED):
            assert np.array_equal(two.ctx.read_buffer(which), one.ctx.read_buffer(which)), (t, which)
        assert all(np.array_equal(two.ctx.get_levels(m), one.ctx.get_levels(m)) for m in (0, 1)), t

    for what in ["fit", "all", "all", "gathered", "all", "node", "all", "gathered", "fit", "all", "all", "capture", "replay", "all", "replay",
                 "gathered", "all", "node", "replay", "replay", "gathered", "all"]:
        t += 1
        grads = [[(rng.standard_t(3, s) * 2.0 ** rng.integers(-3, 3)).astype(np.float32) for s in sizes] for _ in range(K)]
        for m in (two, one):
            m.set_grads(grads)
        torch.cuda.synchronize()
        if what == "capture":
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                two.ctx.quantize_all(two.grad_ptrs(), 77, two.msg[0], None)
            continue
        for m in (two, one):
            if what == "fit":
                m.fit(t)
            elif what == "gathered":
                m.ctx.fit_levels(None, t)
            elif what == "node":
                m.ctx.quantize(1, m.layer_ptrs(m.grad_flat[1]), t, m.msg[0][1], None)
            elif what == "all":
                m.ctx.quantize_all(m.grad_ptrs(), t, m.msg[0], None)
            elif m is two:
                graph.replay()
            else:
                m.ctx.quantize_all(m.grad_ptrs(), 77, m.msg[0], None)
        torch.cuda.synchronize()
        same()
