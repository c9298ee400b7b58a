"""The binding's and the solver's handling of arguments, without a GPU."""
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2505_14371_amd import qoda  # noqa: E402


@pytest.mark.parametrize("has_raw", [True, False])
def test_current_stream_with_and_without_torchs_private_function(monkeypatch, has_raw):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    if has_raw:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 70 + device, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert qoda._stream(None) == (73 if has_raw else 77)
    assert qoda._stream(5) == 5 and qoda._stream(0) is None
    assert qoda._stream(types.SimpleNamespace(cuda_stream=9)) == 9


def test_gradients_are_compared_with_the_parameters_as_they_are():
    """A parameter that was given another size since the solver was made: gradients of the old size are refused."""
    from paper_2505_14371_amd.solver import QODA

    class Grad(torch.Tensor):
        is_cuda = True

    opt = object.__new__(QODA)
    opt.params, opt.K = [torch.zeros(6), torch.zeros(3)], 2
    grads = [[torch.zeros(n).as_subclass(Grad) for n in (6, 3)] for _ in range(2)]
    assert list(opt._check_grads(grads)) == [g.data_ptr() for node in grads for g in node]
    opt.params[1].data = torch.zeros(5)
    with pytest.raises(ValueError):
        opt._check_grads(grads)


def test_native_look_at_the_gradients_leaves_the_rest_to_the_python_one():
    """Nothing on the CPU is accepted, in whatever form it comes, and nothing breaks.  (What else is refused, one cause at a time:
    tests/test_gpu_solver.py.)"""
    import ctypes

    from paper_2505_14371_amd import solver

    if solver._qoda_torch is None:
        from paper_2505_14371_amd import build

        build.build_torch()
        from paper_2505_14371_amd import _qoda_torch as native
    else:
        native = solver._qoda_torch

    class Sub(torch.Tensor):
        is_cuda = True

    params = [torch.nn.Parameter(torch.zeros(4, 3)), torch.zeros(5)]
    out = (ctypes.c_void_p * 4)()
    good = [[torch.zeros(4, 3), torch.zeros(5)] for _ in range(2)]
    for grads in (good, [[g.as_subclass(Sub) for g in node] for node in good], good[:1], [[*good[0], good[0][0]], good[1]], iter(good),
                  [iter(good[0]), good[1]], [[None, None], good[1]], [[1, 2], good[1]], [], None):
        assert native.gather(grads, params, 2, ctypes.addressof(out)) is False
    assert list(out) == [None] * 4
    with pytest.raises(TypeError):
        native.gather(good, params)
    with pytest.raises(TypeError):
        native.gather(good, params, "2", 0)


@pytest.mark.parametrize("why", [ImportError("no torch"), FileNotFoundError("g++"), None])
def test_the_library_is_built_without_the_loops_native_part(monkeypatch, tmp_path, why):
    import subprocess

    from paper_2505_14371_amd import build

    left = tmp_path / "_qoda_torch.so"          # of a build with another torch
    left.write_bytes(b"")
    ran = []

    def run(cmd):
        ran.append(cmd[-1] if build.TORCH_SRC not in cmd else "torch")
        if ran[-1] == "torch":
            raise subprocess.CalledProcessError(1, cmd) if why is None else why

    monkeypatch.setattr(build, "TORCH_LIB", str(left))
    monkeypatch.setattr(build.subprocess, "check_call", run)
    with pytest.warns(UserWarning, match="_qoda_torch.so was not built"):
        assert build.build() == build.LIB
    assert len(ran) == 3 and ran[-1] == "torch" and not left.exists()


def test_a_native_part_built_for_another_torch_is_not_used(monkeypatch):
    import paper_2505_14371_amd as package
    from paper_2505_14371_amd import build, solver

    for has, used in ((types.SimpleNamespace(), False), (types.SimpleNamespace(built_for="2.0.0 cpython-310"), False),
                      (types.SimpleNamespace(built_for=build.built_for()), True)):
        monkeypatch.setattr(package, "_qoda_torch", has, raising=False)
        assert (solver._native_look() is has) == used and (solver._native_look() is None) != used


@pytest.mark.parametrize("symbol, cls, label", [
    ("void qoda::k_quantize<4, true>(qoda::Dev)", "k_quantize", "k_quantize"),
    ("void qoda::k_quantize_b<4, false, 2>(qoda::Dev)", "k_quantize", "k_quantize (no prev)"),
    ("void qoda::k_quantize_small<4, true>(qoda::Dev)", "k_quantize", "k_quantize [with norms and delta]"),
    ("void qoda::k_quantize_held<4, false>(qoda::Dev)", "k_quantize", "k_quantize (no prev) [with norms]"),
    ("void qoda::k_decode<4, 1, false>(qoda::Dev)", "k_decode<true>", "k_decode<true>"),
    ("void qoda::k_decode<4, 4, false>(qoda::Dev)", "k_decode<true>", "k_decode<true> [with step size]"),
    ("void qoda::k_fit_dp<1>(qoda::Dev)", "k_fit_dp", "k_fit_dp [with norms and pooling]"),
    ("void qoda::k_sumsq<true, 2>(qoda::Dev)", "k_sumsq<true>", "k_sumsq<true>")])
def test_profile_summary_knows_the_kernels(symbol, cls, label):
    from paper_2505_14371_amd.harness import profile_summary

    names = [qoda.kernel_name(i) for i in range(qoda.NUM_KERNELS)]
    assert profile_summary._short(symbol) == cls and cls in names
    assert profile_summary._label(symbol) == label
