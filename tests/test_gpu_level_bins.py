"""The table of levels by grid bin and the bucket norms, at the values where they could go wrong: levels in, on and below the
first bin (2^-32), values below it, u = 1 in layers of one pair of blocks; sums of squares next to squares of floats.
Messages and distances, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2505_14371_amd import qoda  # noqa: E402


def gm(*a, **k):
    if not torch.cuda.is_available():
        pytest.fail("a GPU test was selected but no GPU is visible")
    import gpu_harness

    return gpu_harness.GpuModel(*a, **k)


def check(oracle, sizes, lev, grads, scope, kind, separate):
    """Two rounds of every node against the oracle; separate: the kernels one by one instead of the one of small models."""
    K, L, S = len(grads), len(sizes), len(lev)
    m = gm(sizes, [0] * L, [S], K, seed=9, norm_scope=scope, norm_kind=kind)
    m.set_grads(grads)
    m.ctx.set_levels(0, lev)
    if separate:
        m.ctx.profile_enable(["k_delta_finalize"])
    prev = [None] * K
    for t in (1, 2):
        m.quantize_all(t)
        msgs, delta = m.messages(), m.ctx.read_buffer(qoda.BUF_DELTA)
        for k in range(K):
            out = oracle.quantize(sizes, [S] * L, [lev] * L, grads[k], 9, t, k, msg_prev=prev[k], scope=scope, norm_kind=kind)
            assert np.array_equal(msgs[k], out[0]) and delta[k] == out[2], (t, k)
            prev[k] = out[0]
        m.cur, m.have_prev = 1 - m.cur, True


FIRST = np.float32(2.0 ** -32)
LEVELS = {"below": [2.0 ** -40, 0.25], "at": [FIRST, 0.25], "inside": [FIRST * np.float32(1.0625), 0.25], "above": [FIRST * np.float32(1.125), 0.25],
          "two inside": [FIRST * np.float32(1.03), FIRST * np.float32(1.09)], "many below": [2.0 ** -q for q in range(60, 30, -3)],
          "none": [], "edges": [2.0 ** -5, 2.0 ** -4 * 1.125, 0.875], "inside the last": [0.5, 0.99]}


@pytest.mark.parametrize("scope, separate", [(0, False), (0, True), (1, True), (2, False)])
@pytest.mark.parametrize("name", list(LEVELS))
def test_levels_around_the_first_and_last_bin(oracle, name, scope, separate):
    lev = np.array([0.0] + sorted(LEVELS[name]) + [1.0], np.float32)
    rng = np.random.default_rng(len(name))
    sizes = [300, 1, 5000, 513, 2048]
    grads = []
    for k in range(2):
        g = [(rng.choice([-1, 1], s) * 2.0 ** rng.uniform(-45, 0, s)).astype(np.float32) for s in sizes]
        for x in g:
            x[rng.integers(0, x.size, max(1, x.size // 200))] = 1.0     # the norm is near 1: u from 2^-46 to 1
        if k == 1:
            g[0][:] = 0.0
            g[0][130] = -3.0      # alone in its bucket and its layer: u = 1
        grads.append(g)
    check(oracle, sizes, lev, grads, scope, qoda.NORM_L2, separate)


@pytest.mark.parametrize("kind", [qoda.NORM_L2, qoda.NORM_L1, qoda.NORM_LINF])
def test_bucket_norms_next_to_floats(oracle, kind):
    """One, two or four entries in a bucket: sums whose root is a float or lies right beside one, over the exponents of the
    straight-line form and beyond."""
    rng = np.random.default_rng(kind)
    n = 128 * 4096
    x = np.zeros((n // 128, 128), np.float32)
    mant = rng.integers(0, 1 << 23, n // 128)
    mant[::7] = rng.integers(0, 16, mant[::7].size)                     # just above a power of two
    mant[1::7] = (1 << 23) - 1 - rng.integers(0, 16, mant[1::7].size)   # just below
    v = np.ldexp(1.0 + mant / 2.0 ** 23, rng.integers(-62, 62, n // 128)).astype(np.float32)
    v[3::101] = np.ldexp(v[3::101], 1)
    x[:, 5] = v
    x[1::4, 77] = -v[1::4]
    x[2::4, 6:9] = np.float32(2.0 ** -12) * v[2::4, None]               # the root moves by about a unit of its last place
    x[3::4, 100] = np.float32(2.0 ** -11.5) * v[3::4]
    check(oracle, [n], np.array([0.0, 0.1, 0.5, 1.0], np.float32), [[x.reshape(-1)]], qoda.SCOPE_BUCKET, kind, False)


@pytest.mark.parametrize("S", [2, 4, 8, 16, 32, 64, 128, 256])
@pytest.mark.parametrize("walk", [False, True])
def test_both_tables_of_every_width(oracle, S, walk):
    """1700 tiles in the call of both nodes and 850 in each node's own: what one call looks up by grid bin, without a previous message
    up to 6 bits and with it from 9 on, the other looks up by byte.  Levels on bin edges or inside bins."""
    rng = np.random.default_rng(S)
    sizes = [int(x) for x in rng.integers(1, 700, 848)] + [16384 + 77]
    grads = [[(rng.choice([-1, 1], s) * 2.0 ** rng.uniform(-36, 0, s)).astype(np.float32) for s in sizes] for _ in range(2)]
    edge = np.sort(rng.choice(254, S - 2, replace=False)) + 1
    lev = np.concatenate([[0.0], (np.uint32(760) + edge.astype(np.uint32) << 20).view(np.float32), [1.0]]).astype(np.float32)
    if walk and S > 2:
        lev[1:-1] *= np.float32(1.03)
    L = len(sizes)
    want, prev = [[None] * 2, [None] * 2], [None] * 2
    for t in (1, 2):
        for k in range(2):
            want[t - 1][k] = oracle.quantize(sizes, [S] * L, [lev] * L, grads[k], 9, t, k, msg_prev=prev[k])
            prev[k] = want[t - 1][k][0]
    for each in (False, True):
        m = gm(sizes, [0] * L, [S], 2, seed=9)
        assert sum((s + 16383) // 16384 for s in sizes) == 850
        m.set_grads(grads)
        m.ctx.set_levels(0, lev)
        for t in (1, 2):
            (m.quantize_each if each else m.quantize_all)(t)
            msgs, delta = m.messages(), m.ctx.read_buffer(qoda.BUF_DELTA)
            for k in range(2):
                assert np.array_equal(msgs[k], want[t - 1][k][0]) and delta[k] == want[t - 1][k][2], (each, t, k)
            m.cur, m.have_prev = 1 - m.cur, True
