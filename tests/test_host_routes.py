"""Which launches a call makes, seen on the CPU: the library's host side over stand-ins for HIP and the kernels
(tests/host_api_stand_in.cpp), driven through the ordinary binding."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM_INCLUDE = "/opt/rocm/include"


@pytest.fixture(scope="session")
def stand_in(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir(ROCM_INCLUDE):
        pytest.skip("no g++ or no HIP headers")
    lib = str(tmp_path_factory.mktemp("routes") / "libqoda_routes.so")
    cmd = [gxx, "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__",
           "-Wl,-Bsymbolic",       # its own hip functions, also where another library of the process has some
           "-D__align__(n)=__attribute__((aligned(n)))", "-DHIP_SYMBOL(x)=static_cast<const void*>(&x)", "-I" + ROCM_INCLUDE, "-x", "c++",
           os.path.join(HERE, "host_api_stand_in.cpp"), "-o", lib]
    done = subprocess.run(cmd, capture_output=True, text=True)
    assert done.returncode == 0, done.stderr[-4000:]
    return lib


@pytest.fixture()
def routes(stand_in, monkeypatch):
    """make(sizes, ...) -> (context, launches(call) -> names of the launches the call makes)."""
    from paper_2505_14371_amd import qoda

    monkeypatch.setattr(qoda, "_lib", None)
    monkeypatch.setattr(qoda, "LIB_PATH", stand_in)
    lib = qoda.load()
    lib.stand_in_log.restype = ctypes.c_char_p

    class Model:
        def __init__(self, sizes, types=None, points=(8,), K=1, **kw):
            types = [0] * len(sizes) if types is None else types
            self.ctx = qoda.Context(sizes, types, list(points), K, 1, **kw)
            self.K, self.L = K, len(sizes)
            self.grads = [4096] * (K * len(sizes))       # never read: any aligned address will do
            self.msgs, self.prev = [[4096 + 256 * (2 * k + h) for k in range(K)] for h in (0, 1)]
            self.lib = lib
            self.t = 0

        def launches(self, call):
            lib.stand_in_reset()
            call()
            return lib.stand_in_log().decode().split()

        def fit(self, keep=False):
            self.t += 1
            f = self.ctx.fit_levels_keep_norms if keep else self.ctx.fit_levels
            return self.launches(lambda: f(self.grads, self.t, stream=0))

        def histogram(self):
            return self.ctx.read_buffer(qoda.BUF_HIST, stream=0)

    yield Model
    qoda._lib = None


@pytest.mark.parametrize("K, layers, scope", [(2, 3, 0), (3, 11, 0), (2, 3, 1)])   # one kernel after the norm pass; several; vector
class TestHistogramOfTheFit:
    """Every fit counts its own vectors once, whatever happened to the calls before it."""

    def counted_once(self, m):
        h = m.histogram()
        return np.array_equal(h[:, :, 1], np.ones((m.K, m.L), np.uint32)) and h.sum() == m.K * m.L

    def test_repeated(self, routes, K, layers, scope):
        m = routes([100] * layers, K=K, norm_scope=scope)
        assert m.fit().count("zero") == 1            # the first one clears what was allocated
        for _ in range(3):
            assert self.counted_once(m)
            assert "zero" not in m.fit()

    def test_after_a_launch_that_failed(self, routes, K, layers, scope):
        from paper_2505_14371_amd import qoda

        m = routes([100] * layers, K=K, norm_scope=scope)
        n = len(m.fit()) - 1                         # launches of a fit that need not clear
        for at in range(n):
            with pytest.raises(qoda.QodaError):
                m.launches(lambda: (m.lib.stand_in_fail_at(at), m.ctx.fit_levels(m.grads, 50, stream=0)))
            m.fit()
            assert self.counted_once(m), at

    def test_captured(self, routes, K, layers, scope):
        for first_is_captured in (True, False):
            m = routes([100] * layers, K=K, norm_scope=scope)
            if not first_is_captured:
                m.fit()
            m.lib.stand_in_capture(1)
            m.fit()
            m.lib.stand_in_capture(0)
            m.fit()                                  # an eager fit before the first replay
            assert self.counted_once(m)
            m.lib.stand_in_replay()
            assert self.counted_once(m)
            with pytest.raises(Exception):
                m.launches(lambda: (m.lib.stand_in_fail_at(1), m.ctx.fit_levels(m.grads, 50, stream=0)))
            m.lib.stand_in_replay()                  # a replay after a call that failed
            assert self.counted_once(m)
            m.fit()
            assert self.counted_once(m)


@pytest.mark.parametrize("tiles, K, fused", [
    (1, 16, True), (1, 17, False), (8, 16, True), (9, 16, False), (16, 8, True), (17, 8, False), (32, 4, True),
    (40, 1, True), (41, 1, False), (40, 3, True), (64, 64, False), (2, 64, False)])
def test_update_that_computes_its_own_step_size(routes, tiles, K, fused):
    m = routes([16384] * tiles, K=K)
    names = m.launches(lambda: m.ctx.step(m.msgs, m.grads[:tiles], m.grads[:tiles], m.grads[:tiles], 4096, None, 4096, stream=0))
    assert names == (["decode:4"] if fused else ["step_scalars", "decode:1"])
    m.ctx.profile_enable(["k_step_scalars"])
    names = m.launches(lambda: m.ctx.step(m.msgs, m.grads[:tiles], m.grads[:tiles], m.grads[:tiles], 4096, None, 4096, stream=0))
    assert names == ["step_scalars", "decode:1"]


def test_update_of_several_code_widths(routes):
    m = routes([100, 100], types=[0, 1], points=(8, 32))
    names = m.launches(lambda: m.ctx.step(m.msgs, m.grads, m.grads, m.grads, 4096, None, 4096, stream=0))
    assert names == ["step_scalars", "decode:1"]


ONE, SEVERAL = ["norms+hist", "fit_dp:layers"], ["norms+hist", "norm_finalize", "fit_typemax", "fit_pool", "fit_dp:pooled"]


@pytest.mark.parametrize("K, layers, tiles, names", [
    (1, 1, 1, ONE), (1, 8, 1, ONE), (8, 1, 1, ONE), (4, 2, 512, ONE), (1, 1, 4096, ONE),        # up to 8 pairs a type, 4096 tiles
    (1, 9, 1, SEVERAL), (3, 3, 1, SEVERAL), (8, 4, 1, SEVERAL), (4, 2, 513, SEVERAL), (1, 1, 4097, SEVERAL)])
def test_fit_from_vectors(routes, K, layers, tiles, names):
    m = routes([16384 * tiles] + [100] * (layers - 1), K=K)
    m.fit()
    assert m.fit() == names
    m.ctx.profile_enable(["k_fit_pool"])
    assert m.fit() == SEVERAL


@pytest.mark.parametrize("K, layers, one", [(1, 1, True), (4, 8, True), (3, 11, False)])      # 32 pairs, 33
def test_fit_from_gathered_statistics(routes, K, layers, one):
    m = routes([16384 * 3000] + [100] * (layers - 1), K=K, norm_scope=2)
    names = m.launches(lambda: m.ctx.fit_levels(None, 3, stream=0))
    assert names == (["fit_dp:buckets"] if one else ["fit_typemax", "fit_pool_b", "fit_dp:pooled"])


def test_pairs_are_counted_per_type(routes):
    m = routes([100] * 12, types=[l % 2 for l in range(12)], points=(8, 8), K=1)
    m.fit()
    assert m.fit() == ONE


class TestRunsUnderBucketScope:
    """The number of workgroups a node (the length of the table of runs) of the passes that work on runs of tiles."""

    def runs(self, names):
        return {n.split(":")[0]: int(n.split(":")[1]) for n in names if n.split(":")[-1].isdigit()}

    # tiles of a node, K; runs of the quantize pass (all nodes, one node), of the fit from vectors, of the index counts
    @pytest.mark.parametrize("tiles, K, all_nodes, one_node, fit, count", [
        (128, 8, 128, 128, 128, 64), (129, 8, 65, 129, 129, 17), (256, 8, 128, 256, 256, 32), (257, 8, 129, 257, 129, 33),
        (1025, 1, 513, 513, 1025, 129), (1250, 8, 625, 625, 625, 157), (1251, 8, 313, 626, 626, 157), (8192, 8, 2048, 4096, 4096, None)])
    def test_lengths(self, routes, tiles, K, all_nodes, one_node, fit, count):
        m = routes([16384 * tiles - 5], K=K, norm_scope=2)
        assert self.runs(m.launches(lambda: m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0)))["quantize_b"] == all_nodes
        for call in (m.ctx.quantize, m.ctx.quantize_noalloc):
            assert self.runs(m.launches(lambda: call(0, m.grads[:1], 1, m.msgs[0], m.prev[0], stream=0)))["quantize_b"] == one_node
        got = self.runs(m.fit())
        assert got["bucket_max"] == got["bucket_hist"] == fit
        got = self.runs(m.launches(lambda: m.ctx.index_counts(m.msgs, stream=0)))["index_hist"]
        if count is None:       # full runs, with shorter ones at the end of a large table
            T = 2048 // K
            assert got == T + T + T + -(-(tiles - 7 * T) // 8)
        else:
            assert got == count

    def test_runs_end_with_their_layer(self, routes):
        m = routes([16384 * 3, 1, 0, 16384 * 1100], K=1, norm_scope=2)
        assert self.runs(m.launches(lambda: m.ctx.quantize_all(m.grads, 1, m.msgs, None, stream=0)))["quantize_b"] == 2 + 1 + 550

    def test_other_scopes_keep_full_runs(self, routes):
        m = routes([16384 * 100], K=1)
        assert m.launches(lambda: m.ctx.index_counts(m.msgs, stream=0)) == ["zero", "index_hist:13"]


SMALL, LAYERS, VECTOR = ["quantize_small"], ["norms", "norm_finalize", "quantize", "delta"], ["norms", "norm_finalize", "norm_vector", "quantize", "delta"]


@pytest.mark.parametrize("tiles, layers, K, scope, all_nodes, one_node", [
    (1, 1, 1, 0, SMALL, SMALL), (64, 8, 1, 0, SMALL, SMALL), (65, 8, 1, 0, LAYERS, LAYERS), (128, 1, 4, 0, SMALL, SMALL),
    (129, 1, 4, 0, LAYERS, SMALL), (416, 1, 1, 0, SMALL, SMALL), (417, 1, 1, 0, LAYERS, LAYERS), (1, 512, 1, 0, SMALL, SMALL),
    (416, 1, 1, 1, SMALL, SMALL), (417, 1, 1, 1, VECTOR, VECTOR), (6, 64, 1, 1, SMALL, SMALL), (1, 65, 1, 1, VECTOR, VECTOR),
    (200, 2, 2, 1, VECTOR, SMALL)])
def test_one_launch_of_small_models(routes, tiles, layers, K, scope, all_nodes, one_node):
    m = routes([16384 * tiles] * layers, K=K, norm_scope=scope)
    every = lambda: m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0)
    one = lambda: m.ctx.quantize(0, m.grads[:layers], 1, m.msgs[0], m.prev[0], stream=0)
    static = lambda: m.ctx.quantize_noalloc(0, m.grads[:layers], 1, m.msgs[0], None, stream=0)
    separate = VECTOR if scope else LAYERS
    assert m.launches(every) == all_nodes and m.launches(one) == one_node
    assert m.launches(static) == separate                # never: the exchange area is the context's
    m.ctx.profile_enable(["k_quantize", "k_decode<true>"])
    assert m.launches(every) == all_nodes
    m.ctx.profile_enable(["k_delta_finalize"])
    assert m.launches(every) == separate and m.launches(one) == separate


def test_one_launch_is_for_one_code_width_and_computes_norms(routes):
    m = routes([100, 100], types=[0, 1], points=(8, 32))
    call = lambda t=1: m.ctx.quantize_all(m.grads, t, m.msgs, None, stream=0)
    assert m.launches(call) == LAYERS
    m = routes([100, 100])
    m.fit(keep=True)                                     # round 1: the norms are there
    assert m.launches(call) == ["quantize", "delta"]
    assert m.launches(lambda: call(2)) == SMALL and m.launches(call) == SMALL


def test_routes_of_the_sizes_that_the_gpu_tests_compare(routes):
    """tests/test_gpu_small_models.py and tests/test_gpu_fit_paths.py compare a route with the separate kernels.  Here: at their
    sizes it is that route which is taken, or, on the other side of a limit, is not."""
    from test_gpu_small_models import SIZES

    def quantize(m):
        return (m.launches(lambda: m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0)),
                m.launches(lambda: m.ctx.quantize(0, m.grads[:m.L], 1, m.msgs[0], m.prev[0], stream=0)))

    def update(m):
        x = m.grads[:m.L]
        return m.launches(lambda: m.ctx.step(m.msgs, x, x, x, 4096, None, 4096, stream=0))

    # shape: nodes; one launch for all nodes and for one node, under layer and under vector scope; step size in the update
    want = {"ragged": (3, True, True, True, True, True), "edge of a wave pair": (3, True, True, True, True, True),
            "one tile": (3, True, True, True, True, True), "groups beyond 256 tiles": (3, False, True, False, True, False),
            "all 512 tiles": (1, False, False, False, False, False), "513 tiles": (1, False, False, False, False, False),
            "a group of 416 tiles": (1, True, True, False, False, False), "many empty layers": (3, True, True, True, True, True),
            "still more empty layers": (3, True, True, False, False, True)}
    assert set(want) == set(SIZES)
    for shape, (K, *small, fused) in want.items():
        for scope in (0, 1):
            m = routes(SIZES[shape], points=(16,), K=K, norm_scope=scope)
            assert [names == SMALL for names in quantize(m)] == small[2 * scope:2 * scope + 2], (shape, scope)
            assert (update(m) == ["decode:4"]) == fused, shape
    m = routes([1, 2049, 3 * 2048, 2048, 5, 7 * 2048 + 9] * 4, points=(256,), K=5)     # the step sizes of a hundred rounds
    assert update(m) == ["decode:4"]
    for K, layers, layer_scope, bucket_scope in ((1, 1, True, True), (2, 4, True, True), (8, 1, False, True), (3, 3, False, True),
                                                 (4, 8, False, True), (3, 11, False, False), (16, 2, False, True)):
        sizes = [20000] * layers + [0, 16384 * 9 + 5]
        if K == 1:
            sizes[0] = 16384 * 257 + 3
        types = [0] * layers + [0 if layers == 1 else 2, 1]
        points = [8] * (max(types) + 2)
        m = routes(sizes, types=types, points=points, K=K)
        m.fit()
        assert (m.fit() == ONE) == layer_scope, (K, layers)
        m = routes(sizes, types=types, points=points, K=K, norm_scope=2)
        names = m.launches(lambda: m.ctx.fit_levels(None, 3, stream=0))
        assert (names == ["fit_dp:buckets"]) == bucket_scope, (K, layers)


def held(tiles):
    return [f"quantize_held:{tiles}", "delta"]


class TestHeldTiles:
    """Calls that hold their tiles from the norm to the codes."""

    def quantize(self, m, one=False):
        if one:
            return m.launches(lambda: m.ctx.quantize(0, m.grads[:m.L], 1, m.msgs[0], m.prev[0], stream=0))
        return m.launches(lambda: m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0))

    # tiles of a layer, layers, K, scope, grid points; whether all tiles of a call for all nodes are held
    @pytest.mark.parametrize("tiles, layers, K, scope, S, all_nodes", [
        (639, 1, 1, 0, 8, False), (640, 1, 1, 0, 8, True), (1024, 1, 1, 0, 8, True), (1025, 1, 1, 0, 8, False), (409, 1, 40, 0, 8, True),
        (410, 1, 40, 0, 8, False), (682, 1, 3, 0, 8, False), (1023, 1, 2, 0, 8, True), (1024, 2, 1, 0, 8, True), (1024, 3, 1, 0, 8, False),
        (64, 30, 2, 0, 256, True), (65, 48, 1, 0, 256, False), (192, 16, 1, 0, 256, True),
        (193, 10, 1, 0, 256, False), (192, 17, 1, 0, 256, False), (768, 1, 1, 0, 256, True), (769, 1, 1, 0, 256, False), (83, 10, 1, 1, 8, False),
        (84, 10, 1, 1, 8, True), (512, 1, 16, 1, 8, True), (513, 1, 4, 1, 8, False), (513, 1, 3, 1, 8, False), (1024, 1, 3, 1, 8, False),
        (1024, 1, 2, 1, 8, True), (1025, 1, 1, 1, 8, False)])
    def test_lines(self, routes, tiles, layers, K, scope, S, all_nodes):
        m = routes([16384 * tiles] * layers, points=(S,), K=K, norm_scope=scope)
        separate = VECTOR if scope else LAYERS
        assert self.quantize(m) == (held(tiles * layers) if all_nodes else separate)
        assert m.launches(lambda: m.ctx.quantize_noalloc(0, m.grads[:layers], 1, m.msgs[0], None, stream=0)) == separate
        m.ctx.profile_enable(["k_norm_finalize"])
        assert self.quantize(m) == separate

    # tiles of a layer, layers, K, scope, grid points; whether all tiles are held when layers are whole, and when one ends within an octet
    @pytest.mark.parametrize("tiles, layers, K, scope, S, whole, ragged", [
        (513, 1, 2, 0, 8, False, True), (640, 2, 1, 0, 8, True, True), (639, 2, 1, 0, 8, False, True), (256, 1, 5, 0, 8, True, True),
        (257, 1, 4, 0, 8, False, True), (255, 5, 1, 0, 8, True, True), (17, 61, 1, 0, 8, False, True), (17, 68, 1, 0, 8, True, True),
        (16, 65, 1, 0, 8, True, True), (342, 1, 3, 1, 8, False, True), (320, 1, 4, 1, 8, True, True), (682, 1, 3, 0, 8, False, True),
        (683, 1, 3, 0, 8, False, False), (513, 3, 1, 0, 8, False, True), (513, 1, 3, 1, 8, False, False), (700, 1, 2, 1, 8, True, True),
        (1, 769, 1, 0, 256, False, True), (16, 72, 1, 0, 256, False, True), (1, 1153, 1, 0, 256, True, True)])
    def test_ends_of_layers(self, routes, tiles, layers, K, scope, S, whole, ragged):
        separate = VECTOR if scope else LAYERS
        for less, holds in ((0, whole), (2048, whole), (3, ragged), (2047, ragged)):
            m = routes([16384 * tiles] * (layers - 1) + [16384 * tiles - less], points=(S,), K=K, norm_scope=scope)
            assert self.quantize(m) == (held(tiles * layers) if holds else separate), less

    def test_large_layers_among_small_ones(self, routes):
        m = routes([16384 * 100] * 30 + [16384 * 1000], K=1)             # a quarter of the tiles
        assert self.quantize(m) == held(4000)
        m = routes([16384 * 100] * 29 + [16384 * 1000], K=1)
        assert self.quantize(m) == LAYERS
        several = ["norms", "norm_finalize", "quantize_held:2048", "quantize", "delta"]
        m = routes([16384 * 256] * 8 + [16384 * 2000], K=4)              # 8192 small tiles
        assert self.quantize(m) == several and self.quantize(m, one=True) == LAYERS
        assert self.quantize(routes([16384 * 256] * 8 + [16384 * 2000], K=3)) == LAYERS
        assert self.quantize(routes([16384 * 256] * 8 + [16384 * 8192], K=4)) == several
        assert self.quantize(routes([16384 * 256] * 8 + [16384 * 8193], K=4)) == LAYERS

    @pytest.mark.parametrize("sizes, K", [([16384 * 256] * 8 + [16384 * 2000], 4), ([16384 * 400] * 2, 1)])   # small layers held; all
    def test_the_quantizers_time_is_one_launch_a_call(self, routes, sizes, K):
        m = routes(sizes, K=K)
        names = self.quantize(m)
        m.ctx.profile_enable(["k_quantize"])
        for _ in range(3):
            assert self.quantize(m) == names         # the calls that run otherwise
        assert m.ctx.profile_read(stream=0)["k_quantize"][1] == 3

    def test_a_vector_of_several_code_widths(self, routes):
        m = routes([16384 * 450] * 2, types=[0, 1], points=(8, 32), norm_scope=1)
        assert self.quantize(m) == VECTOR
        m = routes([16384 * 450] * 2, types=[0, 1], points=(8, 32))
        assert self.quantize(m) == held(900)

    def test_the_exchange_area_is_zero_when_a_pass_starts(self, routes):
        from paper_2505_14371_amd import qoda

        m = routes([16384 * 400] * 2)
        for at in (0, 1):                                    # the pass, what clears behind it
            with pytest.raises(qoda.QodaError):
                m.launches(lambda: (m.lib.stand_in_fail_at(at), m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0)))
            assert self.quantize(m) == ["zero"] + held(800) and self.quantize(m) == held(800)
        m.lib.stand_in_capture(1)
        assert self.quantize(m) == ["zero"] + held(800)      # for its replays, whatever comes before them
        m.lib.stand_in_capture(0)
        with pytest.raises(qoda.QodaError):
            m.launches(lambda: (m.lib.stand_in_fail_at(1), m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0)))
        m.lib.stand_in_capture(1)
        assert self.quantize(m) == ["zero"] + held(800)      # says nothing about the area now
        m.lib.stand_in_capture(0)
        assert self.quantize(m) == ["zero"] + held(800)

    @pytest.mark.parametrize("one", [False, True])
    def test_replays_after_a_pass_that_failed(self, routes, one):
        """A graph captured while all was well, replayed after an eager pass that failed between its launches."""
        from paper_2505_14371_amd import qoda

        m = routes([16384 * 400] * 2, K=2)
        stale = m.lib.stand_in_stale()
        self.quantize(m)
        m.lib.stand_in_capture(1)
        self.quantize(m, one)
        m.lib.stand_in_capture(0)
        m.lib.stand_in_replay()
        for at in (1, 2):                                    # behind the pass that holds tiles; the second call clears first
            with pytest.raises(qoda.QodaError):
                m.launches(lambda: (m.lib.stand_in_fail_at(at), m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0)))
            m.lib.stand_in_replay()
        assert self.quantize(m) == ["zero"] + held(800)      # all of the area, the rows that the graph does not clear among them
        m.lib.stand_in_replay()
        assert self.quantize(m) == held(800)
        assert m.lib.stand_in_stale() == stale

    @pytest.mark.parametrize("one", [False, True])
    def test_small_layers_beside_others_after_a_launch_that_failed(self, routes, one):
        """Every launch of such a call fails once; a graph captured while all was well is replayed after each failure."""
        from paper_2505_14371_amd import qoda

        m = routes([16384 * 256] * 33 + [16384 * 1025], K=2)
        names = ["norms", "norm_finalize", f"quantize_held:{256 * 33}", "quantize", "delta"]
        stale = m.lib.stand_in_stale()
        assert self.quantize(m, one) == names
        m.lib.stand_in_capture(1)
        assert self.quantize(m, one) == ["zero"] + names
        m.lib.stand_in_capture(0)
        for at in range(5):
            with pytest.raises(qoda.QodaError):
                m.launches(lambda: (m.lib.stand_in_fail_at(at), m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0)))
            m.lib.stand_in_replay()
            assert self.quantize(m, one) == ["zero"] + names and self.quantize(m, one) == names
            m.lib.stand_in_replay()
        assert m.lib.stand_in_stale() == stale

    def test_small_launches_have_an_area_of_their_own(self, routes):
        """One node's 500 tiles in one launch, all nodes' 1000 held: a held pass that fails leaves nothing to the small ones, nor they to clear."""
        from paper_2505_14371_amd import qoda

        m = routes([16384 * 200, 16384 * 300], K=2)
        stale = m.lib.stand_in_stale()
        m.lib.stand_in_capture(1)
        assert self.quantize(m, one=True) == SMALL
        m.lib.stand_in_capture(0)
        with pytest.raises(qoda.QodaError):
            m.launches(lambda: (m.lib.stand_in_fail_at(1), m.ctx.quantize_all(m.grads, 1, m.msgs, m.prev, stream=0)))
        m.lib.stand_in_replay()
        assert self.quantize(m, one=True) == SMALL and self.quantize(m, one=True) == SMALL
        assert self.quantize(m) == ["zero"] + held(500)
        assert m.lib.stand_in_stale() == stale

    def test_sizes_of_the_gpu_tests(self, routes):
        """tests/test_gpu_held_tiles.py compares this route with the separate kernels: at its sizes it is the one that is taken."""
        import test_gpu_held_tiles as g

        def names(sizes, K, scope=0, types=None, points=(16,)):
            return self.quantize(routes(sizes, types=types, points=points, K=K, norm_scope=scope))

        tiles = lambda sizes: sum(-(-s // 16384) for s in sizes)
        for shape, (sizes, K) in g.SIZES.items():
            for S in (16, 130):
                assert (names(sizes, K, points=(S,)) == held(tiles(sizes))) == (S == 16 or "1024" not in shape), (shape, S)
        for sizes, K in g.VECTORS + [g.NODES, g.THREE]:
            assert names(sizes, K, scope=1) == held(tiles(sizes))
        for sizes, K in (g.NODES, g.THREE):
            assert names(sizes, K) == held(tiles(sizes))
        assert names(g.WIDTHS, 1, types=[0, 1, 1, 2, 2], points=(4, 16, 200)) == held(tiles(g.WIDTHS))
        for name, (sizes, K, types, points, _) in g.SOME.items():
            limit = 64 if "nine" in name else 409
            some = [f"quantize_held:{sum(-(-s // 16384) for s in sizes if s <= 16384 * limit)}", "quantize", "delta"]
            assert names(sizes, K, types=types, points=points) == ["norms", "norm_finalize"] + some, name
            m = routes(sizes, types=types, points=points, K=K)
            assert (self.quantize(m, one=True)[2:] == some) == ("one node" in name), name
        assert names(*g.BESIDE)[:3] == ["norms", "norm_finalize", f"quantize_held:{tiles(g.BESIDE[0]) - 1025}"]
