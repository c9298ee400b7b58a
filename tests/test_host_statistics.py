"""Bucket scope: which quantize calls clear the fit's statistics with a launch of their own, and the memory of the two
sets (CPU, over the stand-ins)."""
import ctypes

import numpy as np
import pytest

from paper_2505_14371_amd import qoda
from test_host_routes import routes, stand_in  # noqa: F401  (fixtures)

SWAP = ["quantize_b:3", "delta"]
CLEAR = ["zero_stats"] + SWAP


@pytest.fixture()
def model(routes):  # noqa: F811
    m = routes([16384 * 2, 0, 100], K=2, norm_scope=qoda.SCOPE_BUCKET)
    m.all = lambda: m.launches(lambda: m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0))
    m.one = lambda: m.launches(lambda: m.ctx.quantize(1, m.grads[:3], 1, m.msgs[1], None, stream=0))
    m.gathered = lambda: m.launches(lambda: m.ctx.fit_levels(None, 2, stream=0))
    return m


def test_passes_over_all_nodes_swap_the_sets(model):
    assert [model.all() for _ in range(3)] == [SWAP] * 3
    assert model.one() == CLEAR and model.all() == SWAP            # a node's pass clears its rows of the current set
    assert "zero_stats" in model.fit() and model.all() == SWAP
    model.gathered()
    assert model.all() == SWAP


def test_a_caller_who_times_the_clearing_gets_it(model):
    model.ctx.profile_enable(["k_zero_u32"])
    assert model.all() == CLEAR
    model.ctx.profile_enable([])
    assert model.all() == SWAP


@pytest.mark.parametrize("what", ["all", "one", "gathered", "fit"])
def test_captured_work_keeps_its_set(model, what):
    model.all()
    model.lib.stand_in_capture(1)
    names = getattr(model, what)()
    model.lib.stand_in_capture(0)
    assert what in ("gathered", "fit") or names == CLEAR
    assert [model.all() for _ in range(2)] == [CLEAR] * 2           # it may be replayed at any time


@pytest.mark.parametrize("at", [0, 1])
def test_after_a_launch_that_failed(model, at):
    model.all()
    with pytest.raises(qoda.QodaError):
        model.launches(lambda: (model.lib.stand_in_fail_at(at), model.ctx.quantize_all(model.grads, 1, model.msgs, None, stream=0)))
    assert [model.all() for _ in range(2)] == [CLEAR] * 2


@pytest.mark.parametrize("layers, swaps", [(4096, True), (4097, False)])   # 8192 pairs
def test_large_tables_have_one_set(routes, layers, swaps):  # noqa: F811
    m = routes([10] * layers, K=2, norm_scope=qoda.SCOPE_BUCKET)
    names = m.launches(lambda: m.ctx.quantize_all(m.grads, 1, m.msgs, None, stream=0))
    assert ("zero_stats" not in names) == swaps


def test_both_sets_in_one_histogram_a_pair(routes):  # noqa: F811
    K, L = 2, 300
    lib = routes([10]).lib
    lib.stand_in_allocated.restype = ctypes.c_longlong
    before = lib.stand_in_allocated()
    routes([10] * L, K=K, norm_scope=qoda.SCOPE_BUCKET)
    # 2048 words a pair; all else of it is under 1 KiB: statistic and norm, partial sums, 128 B of each descriptor and of each of the
    # copies of the pointer tables
    assert lib.stand_in_allocated() - before < K * L * (2048 * 4 + 1024) + (1 << 18)


def test_both_sets_read_alike(model):
    want = np.zeros((2, 3, 1024), np.uint64)
    want[:, :, [0, 256]] = 1
    for call in [model.all, model.all, model.all, model.one, model.all, model.all]:
        call()
        assert np.array_equal(model.ctx.read_buffer(qoda.BUF_HIST, stream=0).view(np.uint64), want)
    model.lib.stand_in_capture(1)
    model.all()
    model.lib.stand_in_capture(0)
    for call in [model.lib.stand_in_replay, model.lib.stand_in_replay, model.all, model.lib.stand_in_replay, model.all]:
        call()
        assert np.array_equal(model.ctx.read_buffer(qoda.BUF_HIST, stream=0).view(np.uint64), want)
