"""The native part of the binding against the ctypes calls it stands in front of: the same results, counters and exceptions
whichever of the two takes a call."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2504_04704_amd import lagkv


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
