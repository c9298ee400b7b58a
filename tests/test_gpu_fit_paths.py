"""The level fit that runs in the norm pass and one more kernel (few (node, layer) pairs per type) against the fit that goes
through the separate kernels, which a call takes when their times are asked for or when a type has more pairs.  Histograms,
pooled weights, norms, levels and the messages made with them, bit for bit, over repeated fits.  Which of these sizes take
which route is checked in test_host_routes.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import helpers  # noqa: E402
from paper_2505_14371_amd import qoda  # noqa: E402

SEPARATE = ["k_norm_finalize", "k_fit_typemax", "k_fit_pool"]


def gm(*a, **k):
    if not torch.cuda.is_available():
        pytest.fail("a GPU test was selected but no GPU is visible")
    import gpu_harness

    return gpu_harness.GpuModel(*a, **k)


def state(m, M, scope):
    bufs = [qoda.BUF_SUMSQ, qoda.BUF_POOLED] + ([] if scope == qoda.SCOPE_BUCKET else [qoda.BUF_NORM, qoda.BUF_INV, qoda.BUF_HIST])
    return [m.ctx.read_buffer(b) for b in bufs] + [m.ctx.get_levels(ty) for ty in range(M)] + m.messages() + [m.ctx.status()]


@pytest.mark.parametrize("scope", [qoda.SCOPE_LAYER, qoda.SCOPE_BUCKET])
@pytest.mark.parametrize("kind", [qoda.NORM_L2, qoda.NORM_L1, qoda.NORM_LINF])
@pytest.mark.parametrize("K, layers", [(1, 1), (2, 4), (8, 1), (3, 3), (4, 8), (3, 11), (16, 2)])     # pairs: 8 and 32 are limits
def test_one_kernel_equals_the_separate_ones(K, layers, kind, scope):
    rng = np.random.default_rng([K, layers, kind])
    sizes = [int(s) for s in rng.integers(1, 30000, layers)] + [0, 16384 * 9 + 5]
    sizes[0] = 16384 * 257 + 3 if K == 1 else sizes[0]                          # a layer of more tiles than slots
    types = [0] * layers + [0 if layers == 1 else 2, 1]
    M, L = max(types) + 2, len(sizes)                                           # the last type has no layer
    S = 8
    got = []
    for names in (False, SEPARATE):
        r = np.random.default_rng(5)
        m = gm(sizes, types, [S] * M, K, seed=8, norm_scope=scope, norm_kind=kind)
        m.ctx.profile_enable(names)
        out = []
        for t in range(1, 5):
            g = [[(r.standard_t(3, s) * 2.0 ** t).astype(np.float32) for s in sizes] for _ in range(K)]
            if t == 2:
                for k in range(K):
                    g[k][L - 1][:] = 0.0                                        # a type of zeros keeps its levels
            if t == 3:
                g[0][0][0] = np.inf                                             # so does one with an infinity
            m.set_grads(g)
            if scope == qoda.SCOPE_BUCKET and t > 1:
                m.ctx.fit_levels(None, t)
                m.quantize_all(t)
            else:
                m.ctx.fit_levels_keep_norms(m.grad_ptrs(), t)
                m.quantize_all(t)
            out += state(m, M, scope)
        got.append(out)
        m.ctx.close()
    assert all(np.array_equal(a, b) for a, b in zip(*got))


def test_against_the_oracle(oracle):
    sizes, types, K, S = [5000, 40001, 0, 16384 * 3 + 7, 77], [0, 1, 1, 0, 2], 4, 16
    L, M = len(sizes), 3
    m = gm(sizes, types, [S] * M, K, seed=1)
    levels = [helpers.uniform_levels(S) for _ in range(M)]
    rng = np.random.default_rng(3)
    for t in (1, 2):
        g = [[rng.standard_t(3, s).astype(np.float32) for s in sizes] for _ in range(K)]
        m.set_grads(g)
        m.fit(t)
        levels, hist, pooled, _ = oracle.fit_levels(sizes, types, [S] * M, K, [g[k][l] for k in range(K) for l in range(L)], levels)
        assert np.array_equal(m.ctx.read_buffer(qoda.BUF_HIST).reshape(K * L, -1), np.asarray(hist).reshape(K * L, -1))
        assert np.array_equal(m.ctx.read_buffer(qoda.BUF_POOLED), pooled)
        for ty in range(M):
            assert np.array_equal(m.ctx.get_levels(ty), levels[ty])
