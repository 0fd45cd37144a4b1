"""GPU: the kernel that holds a chunk in registers while the next one's rows arrive through an LDS ring, at the sizes
where it can go wrong: every workgroup size, chunks at and around what its lanes hold, shares that go over from one
stream into the next, lanes and wavefronts without rows of their own."""
import ctypes as C

import pytest
import torch

from paper_2504_04704_amd import lagkv
from tests import parity_util as PU
from tests.test_gpu_parity import gen, run_and_check, say

pytestmark = pytest.mark.gpu

BF, F16, F32 = torch.bfloat16, torch.float16, torch.float32
# streams, scored chunks, D, dtype, L: by the kernel that serves them - wavefronts per tensor and slices a lane holds (0: chunks
# that pass through the ring only) - for rows of up to 64, 128, 256 and 512 bytes.  A wavefront takes 1 KiB of rows a step.
SHAPES = {
    # rows of 64 bytes, of 48 (a lane in four without channels); one chunk more than places; lag of one row
    (1, 8): [(9, 300, 32, BF, 64), (700, 3, 24, F16, 100), (2049, 1, 16, F32, 128), (64, 40, 32, BF, 1), (50, 40, 64, BF, 63), (300, 9, 28, F32, 50),
             (70, 30, 128, F16, 32), (90, 20, 40, F32, 31), (40, 50, 256, BF, 16), (300, 7, 128, F32, 15)],
    # 17 rows in steps of 8, a step and a row short of full, full
    (2, 8): [(300, 5, 128, BF, 33), (70, 16, 80, F16, 63), (41, 27, 96, BF, 64), (33, 70, 64, F32, 57), (90, 12, 24, BF, 129), (37, 15, 16, F32, 256),
             (200, 7, 64, F16, 65), (33, 31, 32, F32, 128), (75, 17, 256, F16, 17), (23, 60, 100, F32, 32)],
    # wavefronts with fewer steps than others, one stream in many shares, many in one
    (4, 8): [(1, 1300, 80, F16, 100), (520, 3, 256, BF, 57), (150, 7, 64, BF, 129), (17, 70, 128, F32, 64), (70, 9, 32, F16, 500), (31, 19, 16, F32, 257),
             (45, 13, 24, F32, 256), (19, 40, 64, F32, 65)],
    # just over eight wavefronts, full
    (8, 8): [(100, 6, 128, F32, 65), (37, 15, 64, F32, 225), (29, 20, 256, BF, 128), (21, 17, 128, F16, 185), (33, 11, 128, BF, 255), (17, 23, 32, F32, 257),
             (30, 9, 24, F32, 512)],
    # 26 and an odd number of steps, all, nearly all
    (4, 32): [(40, 8, 128, BF, 409), (12, 23, 256, F16, 256), (23, 12, 128, F32, 249), (300, 2, 128, F16, 500), (29, 11, 48, F32, 384), (9, 31, 64, F32, 511)],
    # six slots: the fewest steps, an odd number, rows of 64 bytes, the longest chunk of 2-byte rows below 512 KiB
    (4, 0): [(60, 9, 128, F16, 129), (30, 20, 80, BF, 300), (23, 31, 64, BF, 450), (40, 13, 64, F16, 512), (5, 9, 24, BF, 513), (31, 9, 128, BF, 1023),
             (300, 2, 96, F16, 700), (70, 13, 256, BF, 135), (11, 17, 256, F16, 511), (9, 11, 16, F32, 1024), (21, 9, 32, F32, 513), (33, 12, 40, F32, 257),
             (7, 9, 64, F32, 1023), (15, 20, 68, F32, 129), (17, 7, 128, F32, 511)],
    # eight slots
    (8, 0): [(11, 9, 128, BF, 1024), (3, 12, 128, F32, 513), (9, 5, 256, F16, 1000), (13, 7, 64, F32, 1024), (21, 5, 136, BF, 964)],
}


def form(D, esize, L):
    """The library's own choice."""
    lib = lagkv.load()
    lib._ZN5lagkv10ring_holdsEiii.restype = C.c_bool
    waves, holds = lib._ZN5lagkv12ring_threadsEiii(D, esize, L) // 128, lib._ZN5lagkv10ring_holdsEiii(D, esize, L)
    lanes = max(4, 1 << (-(-D * esize // 16) - 1).bit_length())  # of a row
    return waves, 0 if not holds else 8 if L <= 8 * waves * (64 // lanes) else 32


def flat(shapes):
    return [(*x, f) for f, xs in shapes.items() for x in xs]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL])
@pytest.mark.parametrize("streams,n_s,D,dtype,L,kind", flat(SHAPES))
def test_shapes_and_shares_against_the_staged_path(streams, n_s, D, dtype, L, kind, variant):
    say("ring", streams, n_s, D, dtype, L, kind, "variant", variant)
    assert kind is None or form(D, dtype.itemsize, L) == kind
    S, r = (3, 0.3) if L > 3 else (0, 1.0)
    T = S + (n_s + 1) * L + L // 3
    K, V = gen(1, streams, T, D, dtype, seed=streams + L)
    if streams % 2:  # the layout of attention kernels
        K, V = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (K, V))
    assert lagkv.kernel_for(lagkv.params_for(K, S, L, r, variant), T) == "ring_pass_kernel"
    out, _ = run_and_check(K, V, S, L, r, variant=variant, streams=[(0, s) for s in sorted({0, streams // 2, streams - 1})])
    ref = lagkv.score(K, V, S, L, r, variant=variant, launch=lagkv.launch_hint(lagkv.PATH_STAGED))
    assert torch.equal(lagkv.score(K, V, S, L, r, variant=variant), out.scores)
    # two fp32 summation orders of the same sums: a few ulp of a standard deviation of order one
    assert torch.allclose(out.scores, ref, rtol=4e-6, atol=0)
    PU.check_index_invariants(out.idx, T, S, L, out.plan.k, n_s)
    rows = out.idx.long().unsqueeze(-1).expand(-1, -1, -1, D)
    assert torch.equal(out.K, K.gather(2, rows)) and torch.equal(out.V, V.gather(2, rows))
    # the kept set is that of the scores, ties to the lower position
    kept = lagkv.select(out.scores, T, S, L, r)
    assert torch.equal(kept.flatten(2), out.idx[:, :, S:S + n_s * out.plan.k])


# rows of partial slices, on 4-byte addresses: two wavefronts (one lane with channels; a lane short of 64 bytes), four, eight
# with shares over many streams, sixteen with idle wavefronts
PARTIAL = [
    (2050, 1, 4, torch.float32, 64), (40, 30, 30, torch.bfloat16, 111), (300, 5, 100, torch.bfloat16, 57), (1, 900, 126, torch.float16, 128),
    (150, 9, 33, torch.float32, 128), (41, 17, 34, torch.bfloat16, 65), (37, 15, 66, torch.float16, 130), (29, 20, 66, torch.float32, 100),
    (47, 12, 18, torch.bfloat16, 511),
]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL])
@pytest.mark.parametrize("streams,n_s,D,dtype,L", PARTIAL)
def test_partial_slices_and_shares_against_the_staged_path(streams, n_s, D, dtype, L, variant):
    assert D * dtype.itemsize % 4 == 0
    test_shapes_and_shares_against_the_staged_path(streams, n_s, D, dtype, L, None, variant)


# both sides of the rules between the resident, the chunk and the ring kernel
CHOICES = [
    (64, 13, 128, BF, 128), (9, 57, 128, BF, 128), (70, 26, 128, F16, 128), (117, 20, 128, BF, 128), (1, 513, 64, F32, 128), (255, 2, 128, BF, 128),
    (8, 1, 64, BF, 49), (8, 1, 64, BF, 48), (256, 1, 64, F16, 64), (64, 1, 256, BF, 64), (65, 1, 256, BF, 64), (4, 15, 128, F32, 128), (3, 3, 64, F16, 512),
    (256, 1, 50, BF, 64), (257, 1, 50, BF, 64), (33, 1, 16, F32, 512), (257, 1, 16, F32, 257), (256, 1, 32, F16, 300), (4, 75, 64, F32, 1024), (64, 1, 128, BF, 64), (40, 6, 18, BF, 300), (512, 1, 50, BF, 129), (4, 60, 100, BF, 49),
]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL])
@pytest.mark.parametrize("streams,n_s,D,dtype,L", CHOICES)
def test_scores_alone_are_those_of_the_pass(streams, n_s, D, dtype, L, variant):
    """... to the bit, so that lagkv_select on them keeps what lagkv_compress keeps."""
    say("ring, scores alone", streams, n_s, D, dtype, L, "variant", variant)
    S, T = 3, 3 + (n_s + 1) * L + 5
    K, V = gen(1, streams, T, D, dtype, seed=streams + D)
    out, _ = run_and_check(K, V, S, L, 0.25, variant=variant, streams=[(0, 0), (0, streams - 1)])
    scores = lagkv.score(K, V, S, L, 0.25, variant=variant)
    assert torch.equal(scores, out.scores)
    kept = lagkv.select(scores, T, S, L, 0.25)
    assert torch.equal(kept.flatten(2), out.idx[:, :, S:S + n_s * out.plan.k])


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL])
def test_the_error_of_scores_of_long_lags(variant):
    """Against 64 bits, 2-norms.  A score is the sum of two products of an exponential and a reciprocal, each rounded to
    2^-24 of itself at worst; an exponential's own error, that of a standard deviation of order one, is as large.  What a
    chunk's denominator is off by comes on top for all of its tokens, so it may not be off by more than its rounding:
    4.2e-8 in the mean of these shapes then, 4.5e-8 and more with its last additions in 32 bits."""
    errs = []
    for D, dtype, L in [(128, BF, 329), (16, F32, 334), (32, BF, 386), (160, BF, 274), (256, F16, 277), (128, F32, 250), (64, F16, 512),
                        (128, BF, 1000), (64, F32, 700), (128, F16, 200), (80, F16, 450), (96, BF, 600)]:
        streams, n_s, S = 70, 12, 2
        T = S + (n_s + 1) * L
        say("ring, error", D, dtype, L, "variant", variant)
        K, V = gen(1, streams, T, D, dtype, seed=L)
        assert lagkv.kernel_for(lagkv.params_for(K, S, L, 0.25, variant), T) == "ring_pass_kernel"
        got = lagkv.score(K, V, S, L, 0.25, variant=variant).double()
        want = 0
        for x in (K, V):
            x = x.double()[:, :, S:].reshape(1, streams, n_s + 1, L, D)
            own, ref = x[:, :, :-1], x[:, :, 1:] if variant == lagkv.SCORE_LAG else x[:, :, :-1]
            mn, mx = ref.amin(3, keepdim=True), ref.amax(3, keepdim=True)
            want = want + torch.softmax(((own - mn) / (mx - mn)).std(-1), -1)
        errs.append(float((got - want.flatten(2)).norm() / want.norm()))
    assert sum(errs) / len(errs) <= 4.2e-8 and max(errs) <= 5e-8, errs


@pytest.mark.parametrize("D,dtype,L", [(64, torch.bfloat16, 64), (128, torch.bfloat16, 100), (128, torch.float32, 128), (128, torch.float16, 300), (64, torch.bfloat16, 900)])
def test_equal_scores_infinities_and_nan(D, dtype, L):
    """Equal tokens across the edge of the kept set go to the lower positions; a stream with infinities or NaN keeps k
    rows of every chunk, in order, and leaves the streams in the same workgroup what they are."""
    S, n_s, streams = 2, 3, 400
    T = S + (n_s + 1) * L
    say("ring, ties and nan", D, dtype, L)
    K, V = gen(1, streams, T, D, dtype, seed=L)
    K[:, 1, S:S + 2 * L], V[:, 1, S:S + 2 * L] = K[:, 1, S:S + 1], V[:, 1, S:S + 1]
    run_and_check(K, V, S, L, 0.3, streams=[(0, 1), (0, 2)])
    want = lagkv.compress(K, V, S, L, 0.3, want_scores=True)
    K[:, 4, ::3], V[:, 5, ::2, 1], K[:, 6], V[:, 6, 5:] = float("nan"), float("inf"), float("nan"), -float("inf")
    out = lagkv.compress(K, V, S, L, 0.3, want_scores=True)
    PU.check_index_invariants(out.idx, T, S, L, out.plan.k, n_s)
    same = [s for s in range(streams) if s not in (4, 5, 6)]
    for x in ("K", "V", "idx", "scores"):
        assert torch.equal(getattr(out, x)[:, same], getattr(want, x)[:, same])


@pytest.mark.parametrize("D,dtype,L,streams", [(64, torch.bfloat16, 64, 90), (80, torch.float16, 100, 300), (128, torch.float32, 250, 40), (96, torch.bfloat16, 600, 70)])
def test_in_a_captured_graph(D, dtype, L, streams):
    """... replayed three times with eager work between, then on other bytes in the same buffers."""
    S, T = 16, 16 + 9 * L + 17
    K, V = gen(1, streams, T, D, dtype, seed=7)
    want = lagkv.compress(K, V, S, L, 0.25, want_scores=True)
    out = [torch.zeros_like(x) for x in (want.K, want.V, want.idx, want.scores)]

    def call():
        lagkv.compress(K, V, S, L, 0.25, out=(out[0], out[1]), idx_out=out[2], scores_out=out[3])

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for rep in range(4):
        if rep == 3:
            for x, y in zip((K, V), gen(1, streams, T, D, dtype, seed=8)):
                x.copy_(y)
            want = lagkv.compress(K, V, S, L, 0.25, want_scores=True)
        for x in out:
            x.zero_()
        _ = (K.float().sum() + rep).item()
        g.replay()
        torch.cuda.synchronize()
        say("ring graph replay", D, L, rep)
        assert all(torch.equal(x, y) for x, y in zip(out, (want.K, want.V, want.idx, want.scores)))
