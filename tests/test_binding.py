"""The native part of the binding against the ctypes calls it stands in front of: the same results, counters and exceptions
whichever of the two takes a call."""
import ctypes as C
import importlib.util
import warnings

import numpy as np
import pytest
import torch

from paper_2504_04704_amd import build, lagkv


def native():
    lagkv.load()
    assert lagkv._native is not None, "_lagkv_native.so is not built"
    return lagkv._native


def test_forms_that_are_not_plain_are_left_alone():
    n, x = native(), torch.zeros(1, 2, 64, 8)
    assert n.compress(x, x, 1, 8, 0.5, 0, 1, 0, True, False) is None             # no device tensor
    assert n.compress(None, x, 1, 8, 0.5, 0, 1, 0, True, False) is None and n.compress(x) is None
    assert n.append(lagkv.CacheT(), x, 1, 8, 0.5, 0, 1, 0, None, x, x) == -1
    assert n.append(lagkv.CacheT(), x, 1, 8, 0.5, 0, 1, 0, None, None, None) == -1 and n.append() == -1
    with pytest.raises(RuntimeError):
        lagkv.compress(x, x, 1, 8, 0.5)


def test_a_call_that_was_refused_is_not_made_again(monkeypatch):
    class Refuses:
        calls = 0

        def compress(self, *args):
            self.calls += 1
            return lagkv.EHIP

    native()
    monkeypatch.setattr(lagkv, "_native", Refuses())
    monkeypatch.setattr(lagkv, "_prepare", lambda *a: pytest.fail("the ctypes steps"))
    x = torch.zeros(1, 2, 64, 8)
    with pytest.raises(lagkv.LagKVError) as e:
        lagkv.compress(x, x, 1, 8, 0.5)
    assert e.value.status == lagkv.EHIP and "lagkv_compress" in str(e.value) and lagkv._native.calls == 1


def test_a_module_that_does_not_load_is_told_of(monkeypatch):
    """A missing one is not: everything runs through ctypes then.  Nor is a torch without devices one that fails to load."""
    lib = lagkv.load()

    def fails(with_):
        def f(*a):
            raise with_
        monkeypatch.setattr(lagkv.importlib, "import_module", f)

    fails(ImportError("undefined symbol"))
    with pytest.warns(RuntimeWarning, match="undefined symbol"):
        assert lagkv._load_native(lib) is None
    fails(ModuleNotFoundError("No module named '_lagkv_native'"))
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert lagkv._load_native(lib) is None
        monkeypatch.undo()
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
        assert lagkv._load_native(lib) is None


def test_it_builds_without_gcc(monkeypatch, tmp_path):
    which = build.shutil.which
    monkeypatch.setattr(build.shutil, "which", lambda name: None if name in ("g++", "c++") else which(name))
    out = build.build_binding(verbose=False, out_path=str(tmp_path / "_lagkv_native.so"))
    spec = importlib.util.spec_from_file_location("_lagkv_native", out)
    assert importlib.util.module_from_spec(spec).compress() is None


class Sub(torch.Tensor):
    pass


def outcome(f):
    try:
        out = f()
    except Exception as e:  # noqa: BLE001
        return type(e), str(e)
    torch.cuda.synchronize()
    return [x.clone() if isinstance(x, torch.Tensor) else x for x in out]


def equal(a, b):
    if isinstance(a, tuple) or isinstance(b, tuple):
        return a == b
    return len(a) == len(b) and all(torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y for x, y in zip(a, b))


@pytest.mark.gpu
def test_compress_is_the_same_either_way(monkeypatch):
    def fields(c):
        p = c.plan
        return [c.K, c.V, c.idx, c.scores, p.n_chunks, p.n_scored, p.rem, p.k, p.T_out]

    g = torch.Generator(device="cuda").manual_seed(1)
    K, V = (torch.randn(2, 3, 700, 64, device="cuda", generator=g).bfloat16() for _ in range(2))
    B = [x.transpose(1, 2).contiguous().transpose(1, 2) for x in (K, V)]
    odd = [x[..., :50] for x in (K, V)]                                           # (needs a workspace)
    calls = [((K, V, 16, 64, 0.25), {}), ((K, V, 16, 64, 0.25), dict(want_scores=True, want_idx=False)), ((K, V, 16, 512, 0.25), {}),
             ((*B, 0, 100, 0.5), dict(variant=lagkv.SCORE_LOCAL, want_scores=True)), ((*odd, 3, 64, 0.25), dict(variant=lagkv.SCORE_L2)),
             ((K, V, np.int64(16), 64, 1), {}), ((K, V, 16, 64, 0.25), dict(want_idx=1, want_scores=0)), ((K.as_subclass(Sub), V, 16, 64, 0.25), {}),
             ((K.float().requires_grad_(), V.float(), 16, 64, 0.25), {}), ((K, V, 16, 64, 0.25), dict(launch=lagkv.launch_hint(lagkv.PATH_STAGED))),
             # refused
             ((K, V[:, :, :-1], 16, 64, 0.25), {}), ((K, V.half(), 16, 64, 0.25), {}), ((K.double(), V.double(), 16, 64, 0.25), {}),
             ((K[0], V[0], 16, 64, 0.25), {}), ((K[..., ::2], V[..., ::2], 16, 64, 0.25), {}), ((K, V, 16, 64, 0.001), {}), ((K, V, -1, 64, 0.25), {}),
             ((K, V, 1 << 40, 64, 0.25), {}), ((K, V, 16.5, 64, 0.25), {}), ((K, V.cpu(), 16, 64, 0.25), {}), ((K, V, 16, 64, 0.25), dict(variant=7))]
    for n, (args, kw) in enumerate(calls):
        print("[gpu-test] binding, compress", n, flush=True)
        with monkeypatch.context() as m:
            native()
            got = outcome(lambda: fields(lagkv.compress(*args, **kw)))
            m.setattr(lagkv, "_native", None)
            want = outcome(lambda: fields(lagkv.compress(*args, **kw)))
        assert equal(got, want), (n, got, want)


@pytest.mark.gpu
@pytest.mark.parametrize("D,S,L,r", [(25, 3, 64, 0.25), (50, 0, 100, 0.33), (300, 16, 128, 0.5), (64, 2, 50, 0.02)])
def test_the_workspace_of_a_call_is_what_it_asks_for(monkeypatch, D, S, L, r):
    """The size that both ways allocate is the library's own: it takes that and refuses a byte less."""
    launch = lagkv.launch_hint(lagkv.PATH_STAGED)
    for B, T in ((1, S + 2 * L), (3, S + 7 * L + 11)):
        x = torch.randn(B, 2, T, D, device="cuda").half()
        p = lagkv.params_for(x, S, L, r, launch=launch)
        need = lagkv._compress_bytes(p, T, lagkv.plan(p, T))
        print("[gpu-test] binding, workspace", D, B, T, need, flush=True)
        lagkv.compress(x, x, S, L, r, launch=launch, ws=torch.empty(need, dtype=torch.uint8, device="cuda"))
        with pytest.raises(lagkv.LagKVError) as e:
            lagkv.compress(x, x, S, L, r, launch=launch, ws=torch.empty(need - 1, dtype=torch.uint8, device="cuda"))
        assert e.value.status == lagkv.EWORKSPACE
        assert isinstance(native().compress(x, x, S, L, r, 0, 1, launch, True, False), tuple)
        with monkeypatch.context() as m:  # what the library refuses, the native step says itself
            m.setattr(lagkv, "_prepare", lambda *a: pytest.fail("the ctypes steps"))
            with pytest.raises(lagkv.LagKVError) as e:
                lagkv.compress(x, x, S, L, r, launch=lagkv.launch_hint(lagkv.PATH_RESIDENT))
            assert e.value.status == lagkv.ESHAPE
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 50, 25])
def test_append_is_the_same_either_way(monkeypatch, D):
    S, L = 5, 64
    g = torch.Generator(device="cuda").manual_seed(D)
    K, V = (torch.randn(1, 4, S + 5 * L, D, device="cuda", generator=g).bfloat16() for _ in range(2))

    def run(cut):
        c = lagkv.Cache(1, 4, D, S + 4 * L, S, L, 0.25)
        out = []
        for a, b in zip(cut, cut[1:]):
            c.append_and_compress(K[:, :, a:b], V[:, :, a:b])
            out += [c.n_static, c.n_tail, c.n_seen]
        c.append_and_compress(None, None)
        return out + [x.clone() for x in c.view()]

    def refused(k, v):
        c = lagkv.Cache(1, 4, D, 2 * L, S, L, 0.25)
        c.append_and_compress(k, v)
        return [c.n_seen]

    native()
    for n, f in enumerate([lambda: run([0, S + 2 * L, S + 3 * L, S + 3 * L + 1, S + 4 * L]), lambda: run([0, 1, 2, S + 1, S + 2 * L - 1, S + 2 * L]),
                           lambda: run([0, 0, S + 4 * L]), lambda: refused(K, V), lambda: refused(K.half(), V.half()), lambda: refused(K[:, :2], V[:, :2]),
                           lambda: refused(K[0], V[0]), lambda: refused(K[:, :, :9], V[:, :, :8]), lambda: refused(K[:, :, :9].as_subclass(Sub), V[:, :, :9])]):
        print("[gpu-test] binding, append", D, n, flush=True)
        with monkeypatch.context() as m:
            got = outcome(f)
            m.setattr(lagkv, "_native", None)
            want = outcome(f)
        assert equal(got, want), (n, got, want)
