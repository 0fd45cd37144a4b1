"""GPU: the one-shot pass under its own launch choices (nothing hinted), at the sizes where the split of
the work can go wrong: one chunk per segment and several, sink and window rows in one share and in many,
shares of one row, no sink, a window of one lag exactly."""
import pytest
import torch

from paper_2504_04704_amd import lagkv
from tests.test_gpu_parity import gen, run_and_check, say

pytestmark = pytest.mark.gpu

# B, H, chunks, remainder, D, dtype, S, L, r
CASES = [
    (1, 1, 2, 0, 128, torch.bfloat16, 0, 128, 0.25),        # one scored chunk, no sink, a window of one lag
    (1, 2, 3, 127, 128, torch.bfloat16, 1, 128, 0.25),      # shares of the edge rows that do not divide
    (1, 1, 40, 5, 128, torch.bfloat16, 700, 128, 0.25),     # more sink rows than a share holds
    (2, 9, 21, 17, 128, torch.float16, 16, 256, 0.5),       # segments of unequal length
    (5, 67, 9, 30, 64, torch.float32, 16, 128, 0.33),       # more streams than compute units, not a multiple
    (1, 3, 4, 1023, 128, torch.bfloat16, 16, 1024, 0.167),  # a long window
    (3, 100, 5, 3, 96, torch.bfloat16, 4, 64, 0.25),
    (1, 2, 30, 99, 80, torch.float16, 4, 100, 0.33),
]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"B{c[0]}H{c[1]}n{c[2]}m{c[3]}D{c[4]}{str(c[5]).split('.')[-1]}S{c[6]}L{c[7]}")
def test_unhinted_pass_against_oracle(case, variant):
    B, H, n, m, D, dtype, S, L, r = case
    say("launch choice", case, "variant", variant)
    T = S + n * L + m
    K, V = gen(B, H, T, D, dtype, seed=n * 7 + D)
    streams = [(b, h) for b in range(B) for h in range(H)]
    run_and_check(K, V, S, L, r, variant=variant, streams=streams[:2] + streams[-2:] if len(streams) > 4 else streams)
    sc = lagkv.score(K, V, S, L, r, variant=variant)
    torch.cuda.synchronize()
    assert torch.equal(sc, lagkv.compress(K, V, S, L, r, variant=variant, want_scores=True).scores)
