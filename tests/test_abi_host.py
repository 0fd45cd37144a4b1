"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every
symbol the header declares, its partition arithmetic equals Eq. 12 / the oracle, and
every validation error is returned before any device work."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

from oracle import lagkv_oracle as O
from paper_2504_04704_amd import lagkv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(lagkv.lib_path()):
        from paper_2504_04704_amd import build
        build.build_library(verbose=False)
    return lagkv.load()


def test_exports_every_declared_symbol(lib):
    header = open(os.path.join(ROOT, "include", "lagkv.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(lagkv_[a-z_]+)\s*\(", header))
    assert declared == set(lagkv.EXPORTS)
    for name in declared:
        assert getattr(lib, name) is not None


def test_struct_layouts_match_header(tmp_path):
    """The header compiles as plain C and ctypes mirrors its struct layouts."""
    src = tmp_path / "layout.c"
    src.write_text(r"""
#include <stdio.h>
#include <stddef.h>
#include "lagkv.h"
int main(void) {
  printf("%zu %zu %zu %zu %zu %zu %zu %zu %zu %zu\n", sizeof(lagkv_params), offsetof(lagkv_params, r),
         offsetof(lagkv_params, dtype), offsetof(lagkv_params, stride_b), offsetof(lagkv_params, stride_t),
         sizeof(lagkv_plan_t), offsetof(lagkv_plan_t, T_out), sizeof(lagkv_cache),
         offsetof(lagkv_cache, capacity), offsetof(lagkv_cache, n_seen));
  return 0;
}
""")
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe)], check=True)
    got = [int(x) for x in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()]
    P, T, K = lagkv.Params, lagkv.PlanT, lagkv.CacheT
    assert got == [C.sizeof(P), P.r.offset, P.dtype.offset, P.stride_b.offset, P.stride_t.offset,
                   C.sizeof(T), T.T_out.offset, C.sizeof(K), K.capacity.offset, K.n_seen.offset]


def test_plan_equals_eq12_and_oracle(lib):
    rng = np.random.default_rng(0)
    for _ in range(500):
        S = int(rng.integers(0, 40)); L = int(rng.integers(1, 300)); k = int(rng.integers(1, L + 1))
        T = int(rng.integers(1, 5000)); r = (k + 0.5) / L if k < L else 1.0
        p = lagkv.make_params(1, 1, 8, S, L, r)
        pl = lagkv.plan(p, T)
        want = O.plan(T, S, L, r)
        assert (pl.n_chunks, pl.n_scored, pl.rem, pl.k, pl.T_out) == \
            (want["n_chunks"], want["n_scored"], want["rem"], want["k"], want["T_out"])
        if T >= S + 2 * L:
            assert pl.T_out == O.eq12_length(T, S, L, k)
    for T, S, L, rL, n_s, LR in [(1024, 16, 128, 64, 6, 640), (16384, 16, 128, 32, 126, 4288),
                                 (65536, 16, 256, 32, 254, 8640), (131072, 16, 512, 128, 254, 33536),
                                 (32768, 16, 128, 32, 254, 8384), (40960, 16, 128, 32, 318, 10432)]:
        pl = lagkv.plan(lagkv.make_params(4, 8, 128, S, L, rL / L), T)
        assert (pl.k, pl.n_scored, pl.T_out) == (rL, n_s, LR)
    # explicit static part (second pass over a compressed cache is a no-op)
    pl = lagkv.plan(lagkv.make_params(1, 1, 8, 16, 128, 0.25), 4288, 16 + 126 * 32)
    assert pl.n_scored == 0 and pl.T_out == 4288


def _status(fn, *a):
    try:
        fn(*a)
    except lagkv.LagKVError as e:
        return e.status
    return lagkv.OK


def test_keep_for_compression_matches_the_exhaustive_oracle(lib):
    """lagkv_keep_for_compression (closed form + boundary fix-up) against the oracle's
    exhaustive search over rL, on a random grid and at its error cases."""
    import random
    from paper_2504_04704_amd import lagkv
    rnd = random.Random(11)
    for _ in range(2000):
        L = rnd.randint(1, 300); S = rnd.randint(0, 64)
        T = S + 2 * L + rnd.randint(0, 80 * L)
        target = rnd.choice([0.0, rnd.random() * 0.999, O.compression_ratio(T, S, L, rnd.randint(1, L))])
        target = min(max(target, 0.0), 0.999)
        try:
            want = O.keep_for_compression(T, S, L, target)
        except ValueError:
            with pytest.raises(lagkv.LagKVError):
                lagkv.keep_for_compression(T, S, L, target)
            continue
        k, r = lagkv.keep_for_compression(T, S, L, target)
        assert k == want, (T, S, L, target)
        assert O.keep_count(L, r) == k and 0 < r <= 1
    for bad in [(100, 16, 128, 0.5), (10**6, 16, 128, 1.0), (10**6, 16, 128, -0.1), (10**6, -1, 128, 0.5),
                (10**6, 16, 0, 0.5), (10**6, 16, 128, float("nan"))]:
        with pytest.raises(lagkv.LagKVError):
            lagkv.keep_for_compression(*bad)


def test_parameter_validation(lib):
    ok = dict(B=1, H=2, D=64, S=16, L=128, r=0.5)
    def P(**kw):
        d = dict(ok); d.update(kw)
        extra = {k: d.pop(k) for k in ("dtype", "variant", "std_ddof", "strides") if k in d}
        return lagkv.make_params(d["B"], d["H"], d["D"], d["S"], d["L"], d["r"], **extra)
    assert _status(lagkv.plan, P(), 1024) == lagkv.OK
    assert _status(lagkv.plan, P(r=0.0), 1024) == lagkv.EINVAL
    assert _status(lagkv.plan, P(r=1.5), 1024) == lagkv.EINVAL
    assert _status(lagkv.plan, P(r=float("nan")), 1024) == lagkv.EINVAL
    assert _status(lagkv.plan, P(r=0.001), 1024) == lagkv.EINVAL          # floor(r*L) < 1
    assert _status(lagkv.plan, P(L=0), 1024) == lagkv.EINVAL
    assert _status(lagkv.plan, P(S=-1), 1024) == lagkv.EINVAL
    assert _status(lagkv.plan, P(D=1), 1024) == lagkv.ESHAPE              # ddof=1 needs D>=2
    assert _status(lagkv.plan, P(D=1, std_ddof=0), 1024) == lagkv.OK
    assert _status(lagkv.plan, P(std_ddof=2), 1024) == lagkv.EINVAL
    assert _status(lagkv.plan, P(B=0), 1024) == lagkv.ESHAPE
    assert _status(lagkv.plan, P(dtype=7), 1024) == lagkv.EDTYPE
    assert _status(lagkv.plan, P(variant=3), 1024) == lagkv.EDTYPE
    assert _status(lagkv.plan, P(strides=(-1, 0, 0)), 1024) == lagkv.ESHAPE
    assert _status(lagkv.plan, P(), -5) == lagkv.ESHAPE
    assert lib.lagkv_plan(None, 10, -1, C.byref(lagkv.PlanT())) == lagkv.EINVAL
    assert lib.lagkv_plan(C.byref(P()), 10, -1, None) == lagkv.EINVAL
    p = P(); p.launch = -1
    assert _status(lagkv.plan, p, 1024) == lagkv.EINVAL
    p = P(); p.launch = 3 << 2            # 3 wavefronts: not a value lagkv_launch_hint returns
    assert _status(lagkv.plan, p, 1024) == lagkv.EINVAL


def test_calls_reject_bad_arguments_before_touching_the_device(lib):
    p = lagkv.make_params(1, 2, 64, 16, 128, 0.5, lagkv.F32)
    fake = 0x1000                      # never dereferenced: validation fails first
    assert lib.lagkv_score(C.byref(p), None, fake, 1024, fake, None, 0, None) == lagkv.EINVAL
    assert lib.lagkv_score(C.byref(p), fake, fake, 1024, None, None, 0, None) == lagkv.EINVAL
    assert lib.lagkv_score(C.byref(p), fake + 2, fake, 1024, fake, None, 0, None) == lagkv.EINVAL
    assert lib.lagkv_score(C.byref(p), fake, fake, 0, fake, None, 0, None) == lagkv.ESHAPE
    assert lib.lagkv_score(C.byref(p), fake, fake, 100, None, None, 0, None) == lagkv.OK  # below 2L: no-op
    assert lib.lagkv_select(C.byref(p), None, 1024, fake, None) == lagkv.EINVAL
    assert lib.lagkv_select(C.byref(p), fake, 100, None, None) == lagkv.OK
    assert lib.lagkv_compress(C.byref(p), fake, fake, 1024, None, fake, None, None, None, 0, None) == lagkv.EINVAL
    bad_stride = lagkv.make_params(1, 2, 64, 16, 128, 0.5, lagkv.F32, strides=(0, 0, 32))
    assert lib.lagkv_compress(C.byref(bad_stride), fake, fake, 1024, fake, fake, None, None, None, 0,
                              None) == lagkv.ESHAPE
    # positions are int32: a cache of 2^31 rows or more is refused before anything is enqueued
    for T_big in (2 ** 31, 2 ** 40):
        assert lib.lagkv_compress(C.byref(p), fake, fake, T_big, fake, fake, None, None, None, 0, None) == lagkv.ESHAPE
        assert lib.lagkv_score(C.byref(p), fake, fake, T_big, fake, None, 0, None) == lagkv.ESHAPE
        assert lagkv.workspace_bytes(p, T_big) == 0
    # a shape only the three-kernel path serves needs a workspace
    odd = lagkv.make_params(1, 2, 42, 16, 128, 0.5, lagkv.F32)
    need = lagkv.workspace_bytes(odd, 1024)
    assert need > 0 and lagkv.workspace_bytes(p, 1024) == 0
    assert lib.lagkv_compress(C.byref(odd), fake, fake, 1024, fake, fake, None, None, None, 0,
                              None) == lagkv.EWORKSPACE
    assert lib.lagkv_compress(C.byref(odd), fake, fake, 1024, fake, fake, None, None, fake, 64,
                              None) == lagkv.EWORKSPACE
    # forcing the fused kernels on a shape they do not cover is an error, not a fallback
    forced = lagkv.make_params(1, 2, 42, 16, 128, 0.5, lagkv.F32, launch=lagkv.launch_hint(lagkv.PATH_FUSED))
    assert lib.lagkv_compress(C.byref(forced), fake, fake, 1024, fake, fake, None, None, fake, need,
                              None) == lagkv.ESHAPE
    # the staged path asked for by hint needs its workspace even on a fused shape, and says so
    staged = lagkv.make_params(1, 2, 64, 16, 128, 0.5, lagkv.F32, launch=lagkv.launch_hint(lagkv.PATH_STAGED))
    assert lagkv.workspace_bytes(staged, 1024) > 0
    assert lib.lagkv_compress(C.byref(staged), fake, fake, 1024, fake, fake, None, None, None, 0,
                              None) == lagkv.EWORKSPACE
    # L beyond what fits the per-workgroup LDS budget
    huge = lagkv.make_params(1, 1, 64, 0, 1 << 20, 0.5, lagkv.F32)
    assert lib.lagkv_score(C.byref(huge), fake, fake, 1 << 22, fake, None, 0, None) == lagkv.ESHAPE


def test_append_validation(lib):
    p = lagkv.make_params(1, 2, 64, 16, 128, 0.5, lagkv.F32)
    fake = 0x1000
    c = lagkv.CacheT(fake, fake, None, 512, 16, 200, 216)
    assert lib.lagkv_append_and_compress(C.byref(p), C.byref(c), fake, fake, 400, None, 0, None) \
        == lagkv.ECAPACITY
    assert (c.n_static, c.n_tail, c.n_seen) == (16, 200, 216)          # untouched on error
    assert lib.lagkv_append_and_compress(C.byref(p), C.byref(c), None, fake, 4, None, 0, None) == lagkv.EINVAL
    assert lib.lagkv_append_and_compress(C.byref(p), None, fake, fake, 4, None, 0, None) == lagkv.EINVAL
    assert lib.lagkv_append_and_compress(C.byref(p), C.byref(c), fake, fake, -1, None, 0, None) == lagkv.EINVAL
    c2 = lagkv.CacheT(None, fake, None, 512, 0, 0, 0)
    assert lib.lagkv_append_and_compress(C.byref(p), C.byref(c2), fake, fake, 4, None, 0, None) == lagkv.EINVAL


def test_launch_hint_is_a_pure_function(lib):
    """lagkv_launch_hint(_ex) packs its arguments, rejects unknown values, and a call with the
    hint behaves the same however often and in whatever order hints were made (no state)."""
    assert lib.lagkv_launch_hint(0, 0, 0) == 0 and lib.lagkv_launch_hint_ex(0, 0, 0, 0, 0) == 0
    seen = set()
    for path in range(4):
        for waves in (0, 1, 2, 4, 8):
            for seg in (0, 1, 7, 1 << 20):
                v = lib.lagkv_launch_hint(path, waves, seg)
                assert v >= 0 and v == lib.lagkv_launch_hint(path, waves, seg) and v not in seen
                seen.add(v)
                for order in range(4):
                    for sel in range(3):
                        w = lib.lagkv_launch_hint_ex(path, waves, seg, order, sel)
                        assert w >= 0 and (w == v) == (order == 0 and sel == 0)
                        assert _status(lagkv.plan, lagkv.make_params(1, 2, 64, 16, 128, 0.5, launch=w), 1024) == lagkv.OK
    for bad in [(4, 0, 0), (-1, 0, 0), (0, 3, 0), (0, 16, 0), (0, 0, -1), (0, 0, (1 << 20) + 1)]:
        assert lib.lagkv_launch_hint(*bad) == -1
    assert lib.lagkv_launch_hint_ex(0, 0, 0, 4, 0) == -1 and lib.lagkv_launch_hint_ex(0, 0, 0, 0, 3) == -1
    # making other hints in between changes nothing for a call that carries its own
    staged = lagkv.make_params(1, 2, 64, 16, 128, 0.5, lagkv.F32, launch=lagkv.launch_hint(lagkv.PATH_STAGED))
    before = lagkv.workspace_bytes(staged, 4096)
    lagkv.launch_hint(lagkv.PATH_FUSED, 8, 5)
    assert lagkv.workspace_bytes(staged, 4096) == before > 0
    assert lagkv.workspace_bytes(lagkv.make_params(1, 2, 64, 16, 128, 0.5, lagkv.F32), 4096) == 0


def test_path_for_names_the_kernels_of_a_call(lib):
    """lagkv_path_for: rows of 256 bytes with a lag of 128, 256 or 512 are shapes of the register-resident
    kernel (not Eq. 16), other fused shapes of the streaming kernel, the rest of the
    three-kernel path, whichever kernel takes a call of theirs by its size; hints are honoured or refused as lagkv_compress does."""
    mk = lagkv.make_params
    T = 16 + 8 * 512
    for L in (128, 256, 512):
        assert lagkv.path_for(mk(2, 8, 128, 16, L, 0.25, lagkv.BF16), T) == lagkv.PATH_RESIDENT
        assert lagkv.path_for(mk(2, 8, 64, 16, L, 0.25, lagkv.F32), T) == lagkv.PATH_RESIDENT
        assert lagkv.path_for(mk(2, 8, 128, 16, L, 0.25, lagkv.BF16, variant=lagkv.SCORE_LOCAL), T) == lagkv.PATH_RESIDENT
        assert lagkv.path_for(mk(2, 8, 128, 16, L, 0.25, lagkv.BF16, variant=lagkv.SCORE_L2), T) == lagkv.PATH_FUSED
        assert lagkv.path_for(mk(2, 8, 128, 16, L, 0.25, lagkv.BF16, launch=lagkv.launch_hint(lagkv.PATH_FUSED)), T) \
            == lagkv.PATH_FUSED
        assert lagkv.path_for(mk(2, 8, 128, 16, L, 0.25, lagkv.BF16, launch=lagkv.launch_hint(lagkv.PATH_STAGED)), T) \
            == lagkv.PATH_STAGED
    assert lagkv.path_for(mk(2, 8, 128, 16, 100, 0.25, lagkv.BF16), T) == lagkv.PATH_FUSED
    assert lagkv.path_for(mk(2, 8, 128, 16, 512, 0.25, lagkv.F32), T) == lagkv.PATH_FUSED      # rows of 512 bytes
    assert lagkv.path_for(mk(2, 8, 40, 16, 128, 0.25, lagkv.F32), T) == lagkv.PATH_FUSED       # rows of 160 bytes
    assert lagkv.path_for(mk(2, 8, 96, 16, 128, 0.25, lagkv.BF16), T) == lagkv.PATH_FUSED      # rows of 192 bytes
    assert lagkv.path_for(mk(2, 8, 24, 16, 128, 0.25, lagkv.BF16), T) == lagkv.PATH_FUSED      # rows of 48 bytes
    assert lagkv.path_for(mk(2, 8, 16, 16, 128, 0.25, lagkv.BF16), T) == lagkv.PATH_STAGED     # rows of 32 bytes
    assert lagkv.path_for(mk(2, 8, 42, 16, 128, 0.25, lagkv.F32), T) == lagkv.PATH_STAGED      # rows of 168 bytes
    assert lagkv.path_for(mk(2, 8, 264, 16, 128, 0.25, lagkv.BF16), T) == lagkv.PATH_STAGED    # rows of 528 bytes
    for bad in (mk(2, 8, 128, 16, 100, 0.25, lagkv.BF16, launch=lagkv.launch_hint(lagkv.PATH_RESIDENT)),
                mk(2, 8, 42, 16, 128, 0.25, lagkv.F32, launch=lagkv.launch_hint(lagkv.PATH_FUSED))):
        assert lib.lagkv_path_for(C.byref(bad), T) == -lagkv.ESHAPE
    for L, nw in ((1024, 4), (600, 2), (1024, 8), (1024, 0), (512, 4)):          # any workgroup size the hint allows
        hinted = mk(2, 8, 128, 16, L, 0.25, lagkv.BF16, launch=lagkv.launch_hint(lagkv.PATH_FUSED, nw))
        assert lib.lagkv_path_for(C.byref(hinted), 16 + 8 * 1024) == lagkv.PATH_FUSED
    assert lib.lagkv_path_for(C.byref(mk(2, 8, 128, 16, 128, 0.001, lagkv.BF16)), T) == -lagkv.EINVAL
    assert lib.lagkv_path_for(C.byref(mk(2, 8, 128, 16, 128, 0.25, lagkv.BF16)), 0) == -lagkv.ESHAPE


def test_cache_after_compress_and_prefill_rows_follow_eq12(lib):
    """The host calls that keep the partition integers behind the ABI, against the oracle's plan."""
    rng = np.random.default_rng(5)
    for _ in range(300):
        S = int(rng.integers(0, 40)); L = int(rng.integers(1, 200)); k = int(rng.integers(1, L + 1))
        T = int(rng.integers(0, 4000)); r = (k + 0.5) / L if k < L else 1.0
        p = lagkv.make_params(2, 3, 8, S, L, r)
        want = O.plan(T, S, L, r)
        c = lagkv.CacheT(0x1000, 0x1000, None, want["T_out"] + int(rng.integers(0, 3)), 7, 7, 7)
        assert lib.lagkv_cache_after_compress(C.byref(p), T, C.byref(c)) == lagkv.OK
        if want["n_scored"]:
            assert (c.n_static, c.n_tail, c.n_seen) == (S + k * want["n_scored"], L + want["rem"], T)
        else:
            assert (c.n_static, c.n_tail, c.n_seen) == (min(T, S), T - min(T, S), T)
        assert c.n_static + c.n_tail == want["T_out"]
        # chunk-by-chunk prefill: S + 2L rows first, then one lag per call
        empty = lagkv.CacheT(0x1000, 0x1000, None, 10, 0, 0, 0)
        assert lib.lagkv_prefill_rows(C.byref(p), C.byref(empty), 10**9) == S + 2 * L
        assert lib.lagkv_prefill_rows(C.byref(p), C.byref(empty), 5) == min(5, S + 2 * L)
        assert lib.lagkv_prefill_rows(C.byref(p), C.byref(c), 10**9) == (L if T > 0 else S + 2 * L)
        assert lib.lagkv_prefill_rows(C.byref(p), C.byref(c), 0) == 0
    p = lagkv.make_params(1, 1, 8, 16, 128, 0.25)
    small = lagkv.CacheT(0x1000, 0x1000, None, 100, 0, 0, 0)
    assert lib.lagkv_cache_after_compress(C.byref(p), 4096, C.byref(small)) == lagkv.ECAPACITY
    assert (small.n_static, small.n_tail, small.n_seen) == (0, 0, 0)
    assert lib.lagkv_cache_after_compress(C.byref(p), 4096, None) == lagkv.EINVAL
    assert lib.lagkv_cache_after_compress(None, 4096, C.byref(small)) == lagkv.EINVAL
    assert lib.lagkv_prefill_rows(None, C.byref(small), 5) == 0


def test_strerror_and_version(lib):
    for s in range(7):
        assert len(lagkv.strerror(s)) > 1
    assert lagkv.strerror(1234) == "unknown status"
    assert lagkv.version() >= 200


def test_binding_refuses_cpu_tensors():
    import torch
    K = torch.zeros(1, 1, 512, 64)
    with pytest.raises(RuntimeError):
        lagkv.compress(K, K.clone(), 16, 128, 0.5)
    with pytest.raises(RuntimeError):
        lagkv.score(K, K.clone(), 16, 128, 0.5)


def test_kernel_for_names_the_kernel_that_scores(lib):
    """lagkv_kernel_for follows the choice of the call: chunk counts against the places of the kernels, slices per
    lane, Eq. 16, row sizes, hints, and the work items of a grid."""
    def name(streams, D, L, n_s, dtype=lagkv.BF16, variant=lagkv.SCORE_LAG, **kw):
        return lagkv.kernel_for(lagkv.make_params(1, streams, D, 4, L, 1.0, dtype, variant, **kw), 4 + (n_s + 1) * L)
    assert name(8, 128, 512, 1) == "hold_pass_kernel"
    # whole rows: the ring kernel, whatever the number of chunks
    for streams, D, L, n_s in ((1024, 64, 128, 1), (64, 64, 128, 16), (1025, 64, 128, 1), (512, 64, 512, 1), (513, 64, 512, 1),
                               (256, 128, 400, 1), (257, 128, 400, 1), (1, 128, 513, 1)):
        assert name(streams, D, L, n_s) == "ring_pass_kernel"
    # a chunk that it would go over twice, up to two rounds of the chunk kernel
    local = dict(variant=lagkv.SCORE_LOCAL)
    assert name(256, 128, 300, 1, **local) == "chunk_pass_kernel" and name(257, 128, 300, 1, **local) == "ring_pass_kernel"
    assert name(512, 128, 200, 1, **local) == "chunk_pass_kernel" and name(513, 128, 200, 1, **local) == "ring_pass_kernel"
    # Eq. 16 with outputs: half the places
    assert name(256, 128, 128, 1, variant=lagkv.SCORE_L2) == name(128, 128, 512, 1, variant=lagkv.SCORE_L2) == "chunk_pass_kernel"
    assert name(257, 128, 128, 1, variant=lagkv.SCORE_L2) == name(129, 128, 512, 1, variant=lagkv.SCORE_L2) == "split_pass_kernel"
    # rows that are not whole slices: at any count that fits a grid of 512 threads a workgroup, edge copies included
    assert name(100000, 100, 128, 1) == "ring_pass_kernel" and name(100000, 100, 300, 1) == "chunk_pass_kernel"
    assert name((1 << 22) - 1, 5, 2, 1, lagkv.F32) == "ring_pass_kernel" and name(1 << 22, 5, 2, 1, lagkv.F32) == "staged_score_kernel"
    assert name(8, 101, 128, 4) == name(8, 300, 128, 4) == name(8, 100, 513, 4) == "staged_score_kernel"
    # strides of 4-byte multiples, and of odd elements
    assert name(8, 64, 128, 4, strides=(0, 0, 66)) == "ring_pass_kernel" and name(8, 64, 128, 4, strides=(0, 0, 65)) == "staged_score_kernel"
    # any hint keeps it out
    for hint, want in ((lagkv.launch_hint(lagkv.PATH_FUSED), "split_pass_kernel"), (lagkv.launch_hint(lagkv.PATH_STAGED), "staged_score_kernel"),
                       (lagkv.launch_hint(lagkv.PATH_AUTO, 4), "split_pass_kernel"), (lagkv.launch_hint(lagkv.PATH_AUTO, 0, 3), "split_pass_kernel")):
        assert name(8, 64, 128, 4, launch=hint) == want
    assert name(8, 64, 128, 0) == "copy_rows_kernel"
    with pytest.raises(lagkv.LagKVError):
        name(8, 64, 128, 4, launch=lagkv.launch_hint(lagkv.PATH_RESIDENT))


def test_lags_of_128_between_the_resident_and_the_ring_kernel(lib):
    """The sides of the rule: chunks against the ring kernel's places, whole segments against even shares, 256 streams;
    lagkv_path_for names the family of the shape on both."""
    def name(streams, n_s, dtype=lagkv.BF16, variant=lagkv.SCORE_LAG, L=128):
        p, T = lagkv.make_params(1, streams, 64 if dtype == lagkv.F32 else 128, 4, L, 0.25, dtype, variant), 4 + (n_s + 1) * L
        assert lagkv.path_for(p, T) == lagkv.PATH_RESIDENT
        return lagkv.kernel_for(p, T)
    ring, hold = "ring_pass_kernel", "hold_pass_kernel"
    for dtype in (lagkv.BF16, lagkv.F16, lagkv.F32):
        for streams, n_s in ((1, 1), (8, 16), (8, 17), (8, 20), (8, 32), (8, 33), (8, 63), (128, 4), (1, 512)):
            assert name(streams, n_s, dtype) == ring
        assert name(255, 2, dtype) == ring and name(256, 2, dtype) == name(256, 200, dtype, lagkv.SCORE_LOCAL) == hold
        for L in (256, 512):
            assert name(8, 4, dtype, L=L) == hold
    assert name(1, 513, lagkv.F32) == name(9, 57, lagkv.F32, lagkv.SCORE_LOCAL) == hold and name(9, 57) == ring
    # segments of three chunks and of four; longest segments of 1.41 and 1.44, of 1.23 and 1.30 times an even share
    assert name(1, 768) == ring and name(1, 1000) == hold
    assert name(70, 26) == name(65, 30) == ring and name(64, 13) == hold and name(117, 249) == hold
    assert name(64, 13, variant=lagkv.SCORE_LOCAL) == name(117, 249, variant=lagkv.SCORE_LOCAL) == ring


def test_short_calls_between_the_chunk_and_the_ring_kernel(lib):
    """The sides of the rules: chunks, wavefronts, steps, rows that fill their lanes or not, partial slices.  The variant
    decides with them, what is asked for (scores, rows) does not: one name serves lagkv_score and lagkv_compress."""
    def name(streams, D, L, n_s, dtype=lagkv.BF16, variant=lagkv.SCORE_LAG):
        return lagkv.kernel_for(lagkv.make_params(1, streams, D, 4, L, 1.0, dtype, variant), 4 + (n_s + 1) * L)
    ring, chunk, local = "ring_pass_kernel", "chunk_pass_kernel", lagkv.SCORE_LOCAL
    # two wavefronts: steps of 8 rows of 128 bytes, of 4 rows of 208
    assert name(8, 64, 48, 1) == name(8, 104, 24, 32) == name(257, 64, 64, 1) == ring
    assert name(8, 64, 49, 1) == name(8, 104, 25, 32) == name(256, 64, 64, 1) == name(8, 64, 64, 32, variant=local) == chunk
    # four: Eq. 14-15 of full rows and steps, above 64 chunks
    assert name(65, 64, 128, 1) == name(65, 56, 128, 1, variant=local) == name(65, 64, 96, 1, variant=local) == ring
    assert name(64, 64, 128, 1, variant=local) == name(257, 64, 128, 1, variant=local) == ring
    assert name(64, 128, 64, 1, variant=local) == name(8, 32, 256, 2, variant=local) == chunk and name(64, 128, 64, 1) == ring
    assert name(65, 64, 97, 1, variant=local) == name(256, 64, 128, 1, variant=local) == chunk
    # eight, and chunks that pass through or take 32 slices: full rows and steps, 2-byte elements with Eq. 7-8
    for D, L, dtype in ((64, 193, lagkv.BF16), (256, 64, lagkv.F16), (64, 512, lagkv.F16), (256, 256, lagkv.BF16)):
        assert name(64, D, L, 1, dtype) == chunk and name(65, D, L, 1, dtype) == name(64, D - 8, L, 1, dtype) == ring
    assert name(64, 64, 192, 1) == name(64, 32, 256, 1, lagkv.F32) == name(1, 128, 513, 1) == ring
    assert name(64, 32, 256, 1, lagkv.F32, local) == name(256, 64, 256, 1, variant=local) == name(64, 256, 256, 1, variant=local) == chunk
    assert name(257, 64, 256, 1, variant=local) == name(65, 256, 256, 1, variant=local) == ring
    # lags above 256 in eight slices
    for D, L, dtype in ((32, 257, lagkv.BF16), (16, 512, lagkv.F32), (28, 300, lagkv.F32)):
        assert name(256, D, L, 1, dtype) == name(8, D, L, 32, dtype, local) == chunk
        assert name(257, D, L, 1, dtype) == name(257, D, L, 1, dtype, local) == ring
    assert name(8, 48, 256, 1, lagkv.F32) == name(8, 96, 257, 1) == ring
    # streamed by sixteen: more than a chunk a place
    assert name(257, 128, 1024, 1) == name(256, 128, 1024, 1, variant=local) == name(410, 128, 1024, 1, variant=local) == ring
    assert name(257, 128, 1024, 1, variant=local) == name(409, 128, 1024, 1, variant=local) == "split_pass_kernel"
    # sixteen
    assert name(8, 256, 128, 1) == name(8, 128, 128, 1, lagkv.F32, local) == ring
    # partial slices
    assert name(1, 100, 128, 1) == name(512, 50, 129, 2, variant=local) == name(257, 18, 300, 1) == name(257, 50, 64, 1) == ring
    assert name(512, 50, 129, 1, variant=local) == name(256, 18, 300, 1) == name(256, 50, 64, 1) == name(4, 100, 49, 64, variant=local) == chunk
    assert name(1, 50, 48, 1) == name(4, 100, 49, 64) == name(257, 100, 49, 1, variant=local) == ring
