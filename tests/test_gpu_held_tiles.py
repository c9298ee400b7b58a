"""The quantize call that holds its tiles from the norm to the codes (one read of the vectors) against the separate kernels, which
a call runs when their times are asked for: everything bit for bit.  Which route a size takes is checked in test_host_routes.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2505_14371_amd import qoda  # noqa: E402

LAYER, VECTOR = qoda.SCOPE_LAYER, qoda.SCOPE_VECTOR
PARTS = ["k_sumsq<false>", "k_norm_finalize", "k_norm_vector", "k_delta_finalize"]


def gm(*a, **k):
    if not torch.cuda.is_available():
        pytest.fail("a GPU test was selected but no GPU is visible")
    import gpu_harness

    return gpu_harness.GpuModel(*a, **k)


def fill(m, seed):
    """Heavy-tailed vectors, a scale of its own for every (node, layer), drawn on the GPU; the same for every model."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    for k in range(m.K):
        for l, (o, s) in enumerate(zip(m.off, m.sizes)):
            z = torch.randn((2, s), device="cuda:0", generator=gen)
            m.grad_flat[k][int(o): int(o) + s] = z[0] / (z[1].abs() + 1e-3) * 10.0 ** ((7 * k + 3 * l + seed) % 9 - 6)


def call(m, t, each=False):
    """One quantize call of all nodes and what it leaves behind."""
    (m.quantize_each if each else m.quantize_all)(t)
    m.have_prev, m.cur = True, 1 - m.cur
    out = [x.clone() for x in m.msg[1 - m.cur]]
    out += [torch.from_numpy(m.ctx.read_buffer(b)) for b in (qoda.BUF_DELTA, qoda.BUF_SUMSQ, qoda.BUF_NORM, qoda.BUF_INV)]
    return out, m.ctx.status()


def same(a, b):
    return a[1] == b[1] and all(torch.equal(x, y) for x, y in zip(a[0], b[0]))


T = 16384
# layer sizes, K; what the numbers of tiles stand for: a group of every size that a thread of the collector takes (256, 512, 768,
# 1024 tiles), layers of one tile, of one block, empty ones, ragged octets in the first and the second place of a wave
SIZES = {
    "a group of 1024": ([T * 1023 + 5], 1),
    "a group of 768": ([T * 767 + 2047], 1),
    "257 and 500 in a group": ([T * 256 + 2049, 0, T * 500 + 2047, 3], 1),
    # every remainder of a quad, in the first and in the second octet of every wave, and layers of less than two quads
    "ends": ([T * 2 + 2048 * o + r for o in range(8) for r in (1, 2, 3, 4, 6, 255, 1021, 2047)] + [1, 2, 3, 4, 5, 6, 7], 4),
    "small layers": ([1, 0, 255, 2049, 4097, T, T + 1, T * 3 + 6145, T * 40, 300000] * 4 + [0] * 70, 5),
}
VECTORS = [([T * 350 + 5, 0, 9, T * 46 + 2049], 4), ([T, 5, 0, T * 3 - 1] * 60 + [0], 3), ([T * 1000 + 1, 77], 1)]
WIDTHS = [T * 200 + 5, 1000, T * 300, 0, T * 250 + 3]
BESIDE = [T * 1025 - 3, 5, 0, T * 100 + 7, T * 300, 20000], 21     # 8463 small tiles, 29 % of all
# more of small layers beside others: sizes, K, types, grid points, kind of norm
SOME = {
    "several code widths": (*BESIDE, [0, 1, 1, 0, 1, 0], [4, 32], qoda.NORM_L2),
    "the largest would fit": ([T * 1000 - 3, 5, 0, T * 100 + 7, T * 300, 20000], 21, [0] * 6, [16], qoda.NORM_L1),
    "nine bits": ([T * 800 + 1] + [T * 60 + 7] * 10 + [9, 0], 14, [0] * 13, [200], qoda.NORM_LINF),
    "one node is enough": ([T * 1025 + 5] + [T * 256 + 3] * 33 + [0, 77], 2, [0] * 36, [8], qoda.NORM_L2),
}
NODES = [T * 20 + 5, 1, T * 10, 0, T], 30
THREE = [T * 200 + 5, 300, T * 100], 3


@pytest.mark.parametrize("kind, S", [(qoda.NORM_L2, 16), (qoda.NORM_L1, 5), (qoda.NORM_LINF, 130), (qoda.NORM_L2, 2), (qoda.NORM_L2, 3),
                                     (qoda.NORM_L1, 32), (qoda.NORM_LINF, 64), (qoda.NORM_L2, 128)])
@pytest.mark.parametrize("shape", SIZES)
def test_layers(shape, kind, S):
    sizes, K = SIZES[shape]
    ms = [gm(sizes, [l % 2 for l in range(len(sizes))], [S, S], K, seed=9, norm_kind=kind) for _ in range(2)]
    ms[1].ctx.profile_enable(PARTS)
    for m in ms:
        m.ctx.set_levels(1, np.concatenate([[0.0], 2.0 ** -np.arange(S - 2, -1, -1.0)]).astype(np.float32) if S <= 33 else
                         np.linspace(0, 1, S, dtype=np.float32))
    for t in (1, 2, 3):
        for m in ms:
            fill(m, 10 * t)
        assert same(*[call(m, t, each=t == 3) for m in ms]), t
    assert ms[1].ctx.profile_read()["k_norm_finalize"][1] == 2 + K


@pytest.mark.parametrize("kind", [qoda.NORM_L2, qoda.NORM_L1, qoda.NORM_LINF])
@pytest.mark.parametrize("sizes, K", VECTORS)
def test_vectors(sizes, K, kind):
    ms = [gm(sizes, [0] * len(sizes), [16], K, seed=9, norm_scope=VECTOR, norm_kind=kind) for _ in range(2)]
    ms[1].ctx.profile_enable(PARTS)
    for t in (1, 2, 3):
        for m in ms:
            fill(m, 10 * t)
        assert same(*[call(m, t, each=t == 3) for m in ms]), t


def test_several_code_widths():
    ms = [gm(WIDTHS, [0, 1, 1, 2, 2], [4, 16, 200], 1, seed=3) for _ in range(2)]
    ms[1].ctx.profile_enable(PARTS)
    for t in (1, 2):
        for m in ms:
            fill(m, t)
        assert same(*[call(m, t) for m in ms]), t


def test_small_layers_beside_a_large_one():
    sizes, K = BESIDE
    ms = [gm(sizes, [0] * len(sizes), [4], K, seed=3) for _ in range(2)]
    ms[1].ctx.profile_enable(PARTS)
    for t in (1, 2):
        for m in ms:
            fill(m, t)
        assert same(*[call(m, t) for m in ms]), t


@pytest.mark.parametrize("name", SOME)
def test_more_of_small_layers_beside_others(name):
    sizes, K, types, points, kind = SOME[name]
    ms = [gm(sizes, types, points, K, seed=3, norm_kind=kind) for _ in range(2)]
    ms[1].ctx.profile_enable(PARTS)
    for t in (1, 2, 3):
        for m in ms:
            fill(m, t)
        assert same(*[call(m, t, each=t == 3) for m in ms]), t


def test_replays_of_a_captured_call_that_holds_small_layers():
    sizes, K = BESIDE
    replays(sizes, K, [0] * len(sizes), LAYER)


@pytest.mark.parametrize("scope", [LAYER, VECTOR])
def test_workgroups_that_do_the_collecting_themselves(scope):
    """No looks at all, one look and the usual number, in turn, with other vectors each time."""
    sizes, K = NODES
    ms = [gm(sizes, [0] * 5, [16], K, seed=9, norm_scope=scope) for _ in range(2)]
    ms[1].ctx.profile_enable(PARTS)
    for t, tries in enumerate((0, 1024, 1, 0, 1024), 1):
        ms[0].ctx.exchange_tries(tries)
        for m in ms:
            fill(m, t)
        assert same(*[call(m, t) for m in ms]), tries


@pytest.mark.parametrize("sizes, scope", [([T * 1024], LAYER), ([T] * 900, VECTOR)])
def test_a_device_that_others_use_too(sizes, scope):
    """A group that would fill the device, beside a stream of large additions: it does not wait for what cannot start.  (The bound: held 1.6
    and 1.4 times the separate kernels' time; 19 and 4.4 times, with calls of 7 ms, when every workgroup computed all that was missing.)"""
    import time

    m = gm(sizes, [0] * len(sizes), [16], 1, seed=9, norm_scope=scope)
    fill(m, 1)
    gp, calls = qoda.pointer_array(m.grad_ptrs()), 20
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    src = torch.randn(128 << 20, device="cuda:0")
    dst = torch.empty_like(src)
    took = {}
    for names in (PARTS, False):
        m.ctx.profile_enable(names)
        m.ctx.quantize_all(gp, 1, m.msg[0], None)
        torch.cuda.synchronize()
        with torch.cuda.stream(b):
            for _ in range(400):
                torch.add(src, 1.0, out=dst)
        time.sleep(0.003)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record(a)
        for _ in range(calls):
            m.ctx.quantize_all(gp, 1, m.msg[1], m.msg[0], stream=a)
        ev[1].record(a)
        torch.cuda.synchronize()
        took[bool(names)] = ev[0].elapsed_time(ev[1]) / calls, [x.clone() for x in m.msg[1]]
    assert all(torch.equal(x, y) for x, y in zip(took[True][1], took[False][1]))
    assert took[False][0] < 3 * took[True][0], took


@pytest.mark.parametrize("scope", [LAYER, VECTOR])
@pytest.mark.parametrize("bad", [float("inf"), float("nan"), 1e-45])
def test_flags(scope, bad):
    sizes, K = THREE
    seen = []
    for names in (False, PARTS):
        m = gm(sizes, [0] * 3, [8], K, seed=2, norm_scope=scope)
        m.ctx.profile_enable(names)
        for t in (1, 2):
            fill(m, t)
            if t == 1 and bad == 1e-45:
                m.grad_flat[1][int(m.off[1]): int(m.off[1]) + 300] = bad
            elif t == 1:
                m.grad_flat[1][int(m.off[2]) + 7] = bad
            m.quantize_all(1)
            seen.append(m.ctx.status())
        seen.append([x.clone() for x in m.msg[m.cur]])
    assert seen[0] == seen[3] != qoda.OK and seen[1] == seen[4] == qoda.OK
    assert all(torch.equal(a, b) for a, b in zip(seen[2], seen[5]))


@pytest.mark.parametrize("scope", [LAYER, VECTOR])
def test_replays_of_a_captured_call(scope):
    """A captured pass leaves its exchange area ready for the next replay and for eager passes between."""
    sizes, K = THREE
    replays(sizes, K, [0] * 3, scope)


def replays(sizes, K, types, scope):
    ms = [gm(sizes, types, [8], K, seed=3, norm_scope=scope) for _ in range(2)]
    ms[1].ctx.profile_enable(PARTS)

    def one(m):
        m.ctx.quantize_all(m.gp, 5, m.msg[0], m.msg[1])

    for m in ms:
        fill(m, 1)
        m.gp = qoda.pointer_array(m.grad_ptrs())
        one(m)                      # fills the pointer tables
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        one(ms[0])
    for step in range(6):
        for m in ms:
            fill(m, 2 + step)
        if step % 3 == 2:
            one(ms[0])
        else:
            graph.replay()
        one(ms[1])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(ms[0].msg[0], ms[1].msg[0])), step
        assert np.array_equal(ms[0].ctx.read_buffer(qoda.BUF_DELTA), ms[1].ctx.read_buffer(qoda.BUF_DELTA)), step
