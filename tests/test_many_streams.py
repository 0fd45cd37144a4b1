"""GPU: calls of millions of short streams, whose grids come near the 2^32 work items that a launch may have.  A few
streams are repeated over the whole batch, so that the outputs must repeat what a small call gives."""
import pytest
import torch

from paper_2504_04704_amd import lagkv
from tests.test_gpu_parity import gen, say

pytestmark = pytest.mark.gpu
FEW = 1024
LAG = {lagkv.SCORE_LAG: 2, lagkv.SCORE_LOCAL: 5, lagkv.SCORE_L2: 2}  # (two tokens are alike to Eq. 14-15)


def repeated(x, B, H):
    return x.reshape(1, FEW, *x.shape[2:]).repeat(B * H // FEW, 1, 1, 1).view(B, H, *x.shape[2:])


def same_everywhere(big, small):
    small = small.reshape(FEW, -1)
    big = big.reshape(-1, *small.shape)
    return all(torch.equal(part, small.expand_as(part)) for part in big.split(1024))


# 2^24 streams are the most a call takes; 2^22 of the chunk kernel's and 2^23 of a scores-only call's workgroups of
# 512 threads fill a grid, and of the streaming kernel's 128 threads 2^25 (two workgroups per stream)
@pytest.mark.parametrize("B,H,D,variant", [
    (1 << 12, 1 << 12, 12, lagkv.SCORE_LAG),      # rows of 48 bytes: the streaming kernel, ranges of whole batches
    (1, 1 << 24, 12, lagkv.SCORE_L2),             # ... of heads
    (1 << 11, (1 << 13) - 1024, 12, lagkv.SCORE_LOCAL),  # just below the limit
    (1 << 22, 1, 5, lagkv.SCORE_LAG),             # rows of 20 bytes: the chunk kernel's limit
    (1 << 12, 1 << 10, 5, lagkv.SCORE_LOCAL),
])
def test_one_shot_pass_over_millions_of_streams(B, H, D, variant):
    say("millions of streams", B, H, D, "variant", variant)
    S, L, r = 1, LAG[variant], 0.5
    K, V = gen(1, FEW, S + 2 * L + 1, D, torch.float32, seed=D)
    want = lagkv.compress(K, V, S, L, r, variant=variant, want_scores=True)
    out = lagkv.compress(repeated(K, B, H), repeated(V, B, H), S, L, r, variant=variant, want_scores=True)
    torch.cuda.synchronize()
    same = [same_everywhere(getattr(out, x), getattr(want, x)) for x in ("idx", "K", "V")]
    assert same == [True] * 3
    # (another kernel than the small call's may sum in another order: a few ulp of scores of order one)
    assert (out.scores.view(-1, want.scores.numel()) - want.scores.view(1, -1)).abs().max() <= 4e-6 * want.scores.abs().max()


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL])
def test_scores_of_millions_of_streams(variant):
    say("millions of streams, scores", variant)
    K, V = gen(1, FEW, 5, 5, torch.float32, seed=3)
    want = lagkv.score(K, V, 1, 2, 0.5, variant=variant)
    got = lagkv.score(repeated(K, 1 << 13, 1 << 10), repeated(V, 1 << 13, 1 << 10), 1, 2, 0.5, variant=variant)
    torch.cuda.synchronize()
    assert (got.view(-1, want.numel()) - want.view(1, -1)).abs().max() <= 4e-6


@pytest.mark.parametrize("D,variant", [(12, lagkv.SCORE_LOCAL), (4, lagkv.SCORE_LAG)])
def test_a_round_of_millions_of_caches(D, variant):
    """2^23 workgroups of 512 threads fill a grid: the single-round kernel leaves such calls to the others."""
    B, H, S, L, r = 1 << 13, 1 << 10, 1, LAG[variant], 0.5
    say("millions of caches", D, "variant", variant)
    K, V = gen(1, FEW, S + 2 * L, D, torch.float32, seed=D + 1)
    caches = [lagkv.Cache(b, h, D, S + 2 * L, S, L, r, torch.float32, variant=variant) for b, h in ((1, FEW), (B, H))]
    for cache, (k, v) in zip(caches, ((K, V), (repeated(K, B, H), repeated(V, B, H)))):
        cache.append_and_compress(k[:, :, :-1].contiguous(), v[:, :, :-1].contiguous())
        cache.append_and_compress(k[:, :, -1:].contiguous(), v[:, :, -1:].contiguous())
    torch.cuda.synchronize()
    assert caches[0].length == caches[1].length == S + L + L // 2
    same = [same_everywhere(big.contiguous(), small.contiguous()) for small, big in zip(caches[0].view(), caches[1].view())]
    assert same == [True] * 3
