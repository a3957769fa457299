"""The binding's native half (csrc/launch.cpp): it takes plain calls, and hands back, without having done anything, whatever it
does not know, so that the Python path takes or refuses it as it always did."""
import numpy as np
import pytest

import paper_2510_06957_amd as tg
from paper_2510_06957_amd import binding


def test_it_is_built_and_hands_back_what_is_not_on_a_gpu():
    import torch
    t = tg.tcsc_build(np.ones((4, 3), np.int8))
    assert binding._launch is not None
    for entry in range(4):
        assert binding._launch(entry, torch.ones(2, 4), t, None, None, None, None) is None
    for args in ((9, torch.ones(2, 4), t, None, None, None, None), (0, None, t, None, None, None, None),
                 (0, torch.ones(2, 4), None, None, None, None, None), (0, np.ones((2, 4), np.float32), t, None, None, None, None)):
        assert binding._launch(*args) is None
    with pytest.raises(TypeError):
        binding._launch(0, torch.ones(2, 4))
    with pytest.raises(ValueError):
        tg.tstgemm(torch.ones(2, 4), t)
    tg.tcsc_destroy(t)
    t.device_index = 0
    assert binding._launch(0, torch.ones(2, 4), t, None, None, None, None) is None


def test_it_is_not_bound_when_built_for_another_torch(monkeypatch):
    import types

    import torch

    def bind(*addresses):
        bound.append(addresses)

    lib, bound = binding._load(), []
    for version, taken in (("0.0.1", False), (None, False), (torch.__version__, True)):
        fake = types.SimpleNamespace(bind=bind, launch="launch")
        if version is not None:
            fake.torch_version = str(version)
        monkeypatch.setattr(binding, "_launch", None)
        monkeypatch.setattr(tg, "_launch", fake, raising=False)
        binding._bind_launcher(lib)
        assert (binding._launch == "launch") == taken == bool(bound)


def test_the_library_is_built_where_it_cannot_be(monkeypatch, tmp_path, capfd):
    """Without a compiler for it, or without torch's headers, the build goes on, says so, and leaves no older one behind."""
    from paper_2510_06957_amd import build

    def no_torch():
        raise ImportError("no torch")

    monkeypatch.setattr(build, "command", lambda: ["true"])
    for command in (lambda: ["/nonexistent/g++"], lambda: ["false"], no_torch):
        old = tmp_path / "_launch.so"
        old.write_bytes(b"")
        monkeypatch.setattr(build, "LAUNCH", old)
        monkeypatch.setattr(build, "launch_command", command)
        assert build.build() == build.LIB and not old.exists()
        assert "not built" in capfd.readouterr().err
    monkeypatch.setattr(build, "command", lambda: ["false"])
    with pytest.raises(RuntimeError):
        build.build()


@pytest.mark.gpu
@pytest.mark.parametrize("M", [1, 3, 20, 70])
def test_the_same_results_both_ways(M, monkeypatch):
    import torch
    K, N = 130, 70
    rng = np.random.default_rng(970)
    t = tg.tcsc_upload(tg.tcsc_build(rng.integers(-1, 2, (K, N)).astype(np.int8)))
    X, b = torch.randn(M, K, device="cuda"), torch.randn(N, device="cuda")
    one, column = torch.rand(1, device="cuda"), torch.rand(N, device="cuda")
    side = torch.cuda.Stream()
    calls = [lambda: tg.tstgemm(X, t), lambda: tg.tstgemm(X, t, b), lambda: tg.tstgemm(X, t, b, alpha=one),
             lambda: tg.tstgemm(torch.nn.Parameter(X), t, b, alpha=column),
             lambda: tg.tstgemm(X, t, b, torch.empty(M, N, device="cuda")), lambda: tg.tstgemm(X, t, b, stream=side),
             lambda: tg.tstgemm_noalloc(X, t, b, torch.empty(M, N, device="cuda"))]
    if M <= 8:
        calls += [lambda: tg.tstgemm_packed(X, t, b), lambda: tg.tstgemm_signed(X, t, b)]
    torch.cuda.synchronize()
    taken, native_half = [], binding._launch

    def watched(*args):
        taken.append(native_half(*args))
        return taken[-1]

    monkeypatch.setattr(binding, "_launch", watched)
    native = [f() for f in calls]
    torch.cuda.synchronize()
    assert len(taken) == len(calls) and all(done is y for done, y in zip(taken, native))   # each call went that way
    monkeypatch.setattr(binding, "_launch", None)
    for f, y in zip(calls, native):
        z = f()
        torch.cuda.synchronize()
        assert torch.equal(y, z) and y.shape == (M, N) and type(y) is torch.Tensor and not y.requires_grad
    out = torch.empty(M, N, device="cuda")
    monkeypatch.undo()
    assert tg.tstgemm(X, t, b, out) is out


@pytest.mark.gpu
def test_what_was_refused_is_refused():
    import torch
    K, N = 64, 32
    t = tg.tcsc_upload(tg.tcsc_build(np.ones((K, N), np.int8)), forms=tg.FORM_ROWSETS)
    X, b, Y = torch.ones(4, K, device="cuda"), torch.ones(N, device="cuda"), torch.empty(4, N, device="cuda")
    wrong = [dict(X=X.double()), dict(X=X.half()), dict(X=X.t()), dict(X=X[:, ::2]), dict(X=X[0]), dict(X=X.cpu()),
             dict(b=b.double()), dict(b=b[:-1]), dict(b=b.cpu()), dict(b=torch.ones(2 * N, device="cuda")[::2]),
             dict(Y=Y[:3]), dict(Y=Y.t().contiguous().t()), dict(Y=Y.double()), dict(Y=Y.cpu()), dict(alpha=b[:2]),
             dict(alpha=b.double()), dict(alpha=b.cpu())]
    for change in wrong:
        args = dict(X=X, b=b, Y=Y, alpha=None)
        args.update(change)
        with pytest.raises(ValueError):
            tg.tstgemm(args["X"], t, args["b"], args["Y"], alpha=args["alpha"])
    for call, code in ((lambda: tg.tstgemm(X[:, :32].contiguous(), t), -1), (lambda: tg.tstgemm(X[:0], t), -1),
                       (lambda: tg.tstgemm_packed(X, t), -7), (lambda: tg.tstgemm_signed(X, t), -7),
                       (lambda: tg.tstgemm(torch.ones(9, K, device="cuda"), t), -7)):
        with pytest.raises(tg.TstgemmError) as e:
            call()
        assert e.value.code == code
    built = tg.tcsc_build(np.ones((K, N), np.int8))
    with pytest.raises(tg.TstgemmError) as e:
        tg.tstgemm(X, built)
    assert e.value.code == -3
    tg.tcsc_destroy(t)
    with pytest.raises(ValueError):
        tg.tstgemm(X, t)


@pytest.mark.gpu
def test_modes_and_subclasses_see_what_they_saw():
    """A function mode sees the allocation of Y; a tensor of another class goes the long way."""
    import torch
    from torch.overrides import TorchFunctionMode

    seen = []

    class Mode(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    class Other(torch.Tensor):
        pass

    K, N = 64, 32
    t = tg.tcsc_upload(tg.tcsc_build(np.ones((K, N), np.int8)), forms=tg.FORM_ROWSETS)
    X = torch.ones(4, K, device="cuda")
    with Mode():
        Y = tg.tstgemm(X, t)
    assert torch.empty in seen and torch.equal(Y, torch.full((4, N), float(K), device="cuda"))
    assert torch.equal(tg.tstgemm(X.as_subclass(Other), t), Y)


@pytest.mark.gpu
def test_an_error_of_the_gpu_is_raised_at_once(monkeypatch):
    """What the library refuses before it launches anything goes the long way; an error of the GPU does not, so no kernel of the
    call is launched a second time."""
    import ctypes

    import torch

    t = tg.tcsc_upload(tg.tcsc_build(np.ones((64, 32), np.int8)), forms=tg.FORM_ROWSETS)
    X, b, Y = torch.ones(4, 64, device="cuda"), torch.ones(32, device="cuda"), torch.empty(4, 32, device="cuda")
    lib, vp, ci, calls = binding._load(), ctypes.c_void_p, ctypes.c_int, []

    def library(code, *types):
        return ctypes.CFUNCTYPE(ci, *types)(lambda *a: calls.append(code) or code)

    from paper_2510_06957_amd import _launch as native
    for code in (-4, -1):
        plain = library(code, vp, vp, vp, vp, ci, ci, ci, vp)
        prelu = library(code, vp, vp, vp, vp, ci, vp, ci, ci, ci, vp)
        address = [ctypes.cast(f, vp).value for f in (plain, plain, plain, plain, prelu)]
        native.bind(*address, tg.TstgemmError)
        try:
            for entry, name, alpha in ((0, "tstgemm", None), (0, "tstgemm", b), (1, "tstgemm_packed", None), (3, "tstgemm_noalloc", None)):
                calls.clear()
                if code == -4:
                    with pytest.raises(tg.TstgemmError, match=name) as e:
                        native.launch(entry, X, t, b, Y, None, alpha)
                    assert e.value.code == code
                else:
                    assert native.launch(entry, X, t, b, Y, None, alpha) is None
                assert calls == [code]
        finally:
            binding._bind_launcher(lib)
    assert torch.equal(tg.tstgemm(X, t, b, Y), torch.full((4, 32), 65.0, device="cuda"))
