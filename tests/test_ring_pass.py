"""GPU: the kernel that holds a chunk in registers while the next one's rows arrive through an LDS ring, at the sizes
where it can go wrong: every workgroup size, chunks at and around what its lanes hold, shares that go over from one
stream into the next, lanes and wavefronts without rows of their own."""
import pytest
import torch

from paper_2504_04704_amd import lagkv
from tests import parity_util as PU
from tests.test_gpu_parity import gen, run_and_check, say

pytestmark = pytest.mark.gpu

# streams, scored chunks, D, dtype, L.  A wavefront takes 1 KiB of rows a step, a lane 8 slices (32 in the last ones).
SHAPES = [
    # two wavefronts: rows of 64 bytes, of 48 (a lane in four without channels); one chunk more than places; lag of one row
    (9, 300, 32, torch.bfloat16, 64), (700, 3, 24, torch.float16, 100), (2049, 1, 16, torch.float32, 128), (64, 40, 32, torch.bfloat16, 1),
    # four: 17 rows in steps of 8, a step and a row short of full, full
    (300, 5, 128, torch.bfloat16, 33), (70, 16, 80, torch.float16, 63), (41, 27, 96, torch.bfloat16, 64), (33, 70, 64, torch.float32, 57),
    # eight: wavefronts with fewer steps than others, one stream in many shares, many in one
    (1, 1300, 80, torch.float16, 100), (520, 3, 256, torch.bfloat16, 57), (150, 7, 64, torch.bfloat16, 129), (17, 70, 128, torch.float32, 64),
    # sixteen: just over eight, full
    (100, 6, 128, torch.float32, 65), (37, 15, 64, torch.float32, 225), (29, 20, 256, torch.bfloat16, 128), (40, 13, 64, torch.float16, 512),
    # 32 slices: 26 and an odd number of steps, all, nearly all
    (40, 8, 128, torch.bfloat16, 409), (12, 23, 256, torch.float16, 256), (23, 12, 128, torch.float32, 249), (300, 2, 128, torch.float16, 500),
    # chunks that pass through the ring only: eight wavefronts, six slots - the fewest steps, an odd number, rows of 64 bytes, the
    # longest chunk of 2-byte rows below 512 KiB - and sixteen, eight slots
    (60, 9, 128, torch.float16, 129), (30, 20, 80, torch.bfloat16, 300), (23, 31, 64, torch.bfloat16, 450), (5, 9, 24, torch.bfloat16, 513),
    (31, 9, 128, torch.bfloat16, 1023), (300, 2, 96, torch.float16, 700), (11, 9, 128, torch.bfloat16, 1024), (3, 12, 128, torch.float32, 513), (9, 5, 256, torch.float16, 1000),
]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL])
@pytest.mark.parametrize("streams,n_s,D,dtype,L", SHAPES)
def test_shapes_and_shares_against_the_staged_path(streams, n_s, D, dtype, L, variant):
    say("ring", streams, n_s, D, dtype, L, "variant", variant)
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
    (23, 12, 18, torch.bfloat16, 511),
]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL])
@pytest.mark.parametrize("streams,n_s,D,dtype,L", PARTIAL)
def test_partial_slices_and_shares_against_the_staged_path(streams, n_s, D, dtype, L, variant):
    assert D * dtype.itemsize % 4 == 0
    test_shapes_and_shares_against_the_staged_path(streams, n_s, D, dtype, L, variant)


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
