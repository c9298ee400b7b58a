"""The bucket-scope quantize pass where its paths part: weights within and above the low part of the shared-memory
histogram, octets with and without coordinates in raw magnitude bin 0, levels on and inside the bins of the search
table, runs of one tile and of two.  Messages, distances, gathered statistics and the levels fitted from them, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import helpers  # noqa: E402
from paper_2505_14371_amd import qoda  # noqa: E402

BUCKET = qoda.SCOPE_BUCKET


def gm(*a, **k):
    if not torch.cuda.is_available():
        pytest.fail("a GPU test was selected but no GPU is visible")
    import gpu_harness

    return gpu_harness.GpuModel(*a, **k)


def values(kind, n, rng):
    if kind == "equal":          # all buckets weigh about the same: every weight has bits above the low part
        return rng.standard_normal(n).astype(np.float32)
    x = rng.standard_t(3, n).astype(np.float32)
    if kind == "sparse":         # zeros, values of raw magnitude bin 0 and whole buckets of zeros
        x[rng.random(n) < 0.3] = 0.0
        x[rng.random(n) < 0.01] = np.float32(2.0 ** -130)
        x[: min(n, 700)] = 0.0
    if kind == "spiky" and n > 5:   # one bucket outweighs the others by far: low parts only
        x[n // 2] = 1e4
    return x


def check(oracle, m, sizes, S, K, grads, nodes, irregular):
    L = len(sizes)
    lev = np.sort(np.random.default_rng(S).uniform(0.01, 0.9, S - 2)) if irregular else 2.0 ** np.arange(2 - S, 0)
    lev = np.concatenate([[0.0], lev, [1.0]]).astype(np.float32)
    m.set_grads(grads)
    m.fit(1)                                             # gives the passes their weight scale
    flat = [grads[k][l] for k in range(K) for l in range(L)]
    exps = None
    if len(nodes) == K:
        levels, _, _, _ = oracle.fit_levels(sizes, [0] * L, [S], K, flat, [helpers.uniform_levels(S)], scope=BUCKET)
        b0 = np.stack([oracle.quantize(sizes, [S] * L, [levels[0]] * L, grads[k], 31, 0, k, scope=BUCKET,
                                       stats_exp=[oracle.TYPE_SKIP] * L)[5] for k in range(K)])
        _, _, exps, _ = oracle.fit_from_stats([0] * L, [S], K, np.zeros((K, L, 257), np.uint64), b0, [oracle.TYPE_SKIP], levels)
    m.ctx.set_levels(0, lev)
    prev = [None] * K
    for t in (1, 2):
        m.quantize_all(t)
        msgs, delta = m.messages(), m.ctx.read_buffer(qoda.BUF_DELTA)
        hist, bmax = np.zeros((K, L, 257), np.uint64), np.zeros((K, L))
        for k in nodes:
            kw = {} if exps is None else {"stats_exp": [int(exps[0])] * L}
            out = oracle.quantize(sizes, [S] * L, [lev] * L, grads[k], 31, t, k, msg_prev=prev[k], scope=BUCKET, **kw)
            assert np.array_equal(msgs[k], out[0]) and delta[k] == out[2], (t, k)
            prev[k] = out[0]
            if exps is not None:
                hist[k], bmax[k] = out[4], out[5]
        m.cur, m.have_prev = 1 - m.cur, True
    assert m.ctx.status() == qoda.OK
    if exps is not None:
        m.ctx.fit_levels(None, 3)
        levels, pooled, _, _ = oracle.fit_from_stats([0] * L, [S], K, hist, bmax, exps, [lev])
        assert np.array_equal(m.ctx.read_buffer(qoda.BUF_POOLED), pooled)
        assert np.array_equal(m.ctx.get_levels(0), levels[0])


@pytest.mark.parametrize("irregular", [False, True])
@pytest.mark.parametrize("kind", ["equal", "spiky", "sparse"])
@pytest.mark.parametrize("S", [4, 16, 129])
def test_small_models(oracle, S, kind, irregular):
    sizes, K = [1, 129, 2047, 2049, 16385, 0, 3 * 16384 + 4100], 2
    rng = np.random.default_rng([S, len(kind)])
    grads = [[values(kind, s, rng) for s in sizes] for _ in range(K)]
    check(oracle, gm(sizes, [0] * len(sizes), [S], K, seed=31, norm_scope=BUCKET), sizes, S, K, grads, range(K), irregular)


def test_runs_of_two_tiles(oracle):
    """4160 tiles over all nodes; two nodes are compared."""
    sizes, K, S = [16384 * 130 + 5, 2049, 16384 * 127 + 9000], 16, 8
    rng = np.random.default_rng(8)
    base = [values("spiky", s, rng) for s in sizes]
    grads = [[np.roll(b, 77 * k) for b in base] for k in range(K)]
    check(oracle, gm(sizes, [0] * 3, [S], K, seed=31, norm_scope=BUCKET), sizes, S, K, grads, (0, 15), False)


def test_runs_of_four_tiles_equal_single_ones():
    """10 k tiles over all nodes in one call (runs of four, some cut short by the end of a layer) against a call for every
    node (single tiles): messages, distances and gathered statistics."""
    sizes, K = [16384 * 638 + 5, 2049, 16384], 16
    a, b = [gm(sizes, [0] * 3, [16], K, seed=3, norm_scope=BUCKET) for _ in range(2)]
    g = torch.Generator(device="cuda")
    for k in range(K):
        g.manual_seed(k)
        z = torch.randn(a.flat_len, device="cuda", generator=g)
        for m in (a, b):
            m.grad_flat[k].copy_(z ** 3)
    for m in (a, b):
        m.fit(1)
    for t in (1, 2):
        a.quantize_all(t)
        b.quantize_each(t)
        assert np.array_equal(a.ctx.read_buffer(qoda.BUF_DELTA), b.ctx.read_buffer(qoda.BUF_DELTA))
        assert np.array_equal(a.ctx.read_buffer(qoda.BUF_SUMSQ), b.ctx.read_buffer(qoda.BUF_SUMSQ))
        assert np.array_equal(a.ctx.read_buffer(qoda.BUF_HIST), b.ctx.read_buffer(qoda.BUF_HIST))
        for x, y in zip(a.msg[a.cur], b.msg[b.cur]):
            assert torch.equal(x, y)
        for m in (a, b):
            m.cur, m.have_prev = 1 - m.cur, True


@pytest.mark.parametrize("irregular", [False, True])
@pytest.mark.parametrize("kind", ["equal", "spiky", "sparse"])
@pytest.mark.parametrize("S", [4, 16, 129])
def test_small_layers_and_short_last_octets(oracle, S, kind, irregular):
    """Octets of one pair of blocks and of two, layers of one octet (fewer copies of the histogram) and of one octet more."""
    sizes, K = [50, 256, 257, 511, 512, 513, 1024, 2048, 2048 + 1, 2048 + 512, 2048 + 513, 4096, 16384 + 300], 2
    rng = np.random.default_rng([S, len(kind), 1])
    grads = [[values(kind, s, rng) for s in sizes] for _ in range(K)]
    check(oracle, gm(sizes, [0] * len(sizes), [S], K, seed=31, norm_scope=BUCKET), sizes, S, K, grads, range(K), irregular)
