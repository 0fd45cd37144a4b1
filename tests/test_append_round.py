"""GPU: the append under its own launch choices (nothing hinted): the single-round kernel and the plain append, at
the sizes where they can go wrong - the border between cached and new rows anywhere, both ranges of the
selection, chunks that fill a lane's registers and chunks of a few rows, rows of partial slices, a sink that
fills in the same call - against the oracle on the whole history."""
import pytest
import torch

from paper_2504_04704_amd import lagkv
from tests.test_gpu_parity import VARIANT_NAME, gen, oracle_history_check, say

pytestmark = pytest.mark.gpu

SHAPES = [
    # L, D, dtype, r
    (3, 128, torch.bfloat16, 0.67),
    (46, 64, torch.float32, 0.25),
    (128, 128, torch.bfloat16, 0.25),       # 8 slices a lane, all full
    (130, 128, torch.float16, 0.99),        # 16 slices, the last two mostly past the end
    (256, 128, torch.bfloat16, 0.25),       # 16 slices: the reference rows stay in registers
    (257, 128, torch.bfloat16, 0.125),      # 32 slices: they are read again; histogram selection
    (512, 128, torch.bfloat16, 1.0),
    (100, 256, torch.bfloat16, 0.33),
    (500, 80, torch.float16, 0.3),
    (128, 100, torch.bfloat16, 0.25),       # rows of 200 bytes
    (33, 6, torch.float32, 0.5),            # rows of 24 bytes
    (64, 130, torch.float16, 0.25),         # rows of 260 bytes
    (40, 126, torch.float32, 0.1),
]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("L,D,dtype,r", SHAPES)
def test_single_round_append_with_the_border_anywhere(L, D, dtype, r, variant):
    S = 5
    for n_tail, n_new in [(0, 2 * L), (1, 3 * L - 2), (L - 1, L + 1), (L, L), (L + 1, L - 1), (2 * L - 1, 1), (2 * L - 1, L),
                          (L + 2, 2 * L - 3)]:
        say("append round", L, D, dtype, "variant", variant, "tail", n_tail, "new", n_new)
        T = S + n_tail + n_new
        Kh, Vh = gen(1, 3, T, D, dtype, seed=L * 7 + n_tail)
        cache = lagkv.Cache(1, 3, D, T + 4, S, L, r, dtype=dtype, variant=variant, track_positions=True)
        cache.append_and_compress(Kh[:, :, :S + n_tail], Vh[:, :, :S + n_tail])
        assert cache.n_static == S and cache.n_tail == n_tail
        cache.append_and_compress(Kh[:, :, S + n_tail:], Vh[:, :, S + n_tail:])
        torch.cuda.synchronize()
        oracle_history_check(cache, Kh, Vh, S, L, r, VARIANT_NAME[variant])


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("L,D,dtype", [(64, 128, torch.bfloat16), (300, 128, torch.float16), (50, 100, torch.bfloat16)])
def test_the_sink_fills_and_a_chunk_completes_in_one_call(L, D, dtype, variant):
    """... from an empty cache and from a sink that already holds rows; a transposed view as the new rows."""
    for S, held in [(16, 0), (16, 9), (40, 39), (700, 1)]:
        say("sink", S, held, L, D, dtype, "variant", variant)
        T = S + 2 * L + 7
        Kh, Vh = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in gen(2, 2, T + 3 * L, D, dtype, seed=S + held))
        caches = [lagkv.Cache(2, 2, D, T + 3 * L, S, L, 0.25, dtype=dtype, variant=variant, track_positions=pos)
                  for pos in (True, False)]
        for cache in caches:
            t = 0
            for n in [held, T - held, 1, L - 8, 0, L, 3]:     # one round, plain rows, one round, none, one round, plain
                if n:
                    cache.append_and_compress(Kh[:, :, t:t + n], Vh[:, :, t:t + n])
                else:
                    cache.append_and_compress(None, None)
                t += n
        torch.cuda.synchronize()
        oracle_history_check(caches[0], Kh[:, :, :t], Vh[:, :, :t], S, L, 0.25, VARIANT_NAME[variant])
        n = caches[0].length
        assert caches[1].length == n
        assert torch.equal(caches[0].K[:, :, :n], caches[1].K[:, :, :n])
        assert torch.equal(caches[0].V[:, :, :n], caches[1].V[:, :, :n])


@pytest.mark.parametrize("D,dtype", [(128, torch.bfloat16), (100, torch.float16), (13, torch.bfloat16), (4, torch.float32), (127, torch.float32)])
def test_plain_append_keeps_what_lies_around_it(D, dtype):
    """Rows that complete no chunk: only their own places change."""
    say("plain append", D, dtype)
    Kh, Vh = gen(3, 5, 90, D, dtype, seed=D)
    cache = lagkv.Cache(3, 5, D, 100, 4, 64, 0.25, dtype=dtype)
    cache.K.fill_(7), cache.V.fill_(7), cache.pos.fill_(-7)
    for a, b in [(0, 3), (3, 4), (4, 37), (37, 90)]:
        cache.append_and_compress(Kh[:, :, a:b], Vh[:, :, a:b])
    torch.cuda.synchronize()
    K, V, pos = cache.view()
    assert torch.equal(K, Kh) and torch.equal(V, Vh)
    assert torch.equal(pos, torch.arange(90, dtype=torch.int32, device=pos.device).expand(3, 5, 90))
    assert bool((cache.K[:, :, 90:] == 7).all()) and bool((cache.V[:, :, 90:] == 7).all()) and bool((cache.pos[:, :, 90:] == -7).all())


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("L,D,dtype", [(64, 128, torch.bfloat16), (160, 96, torch.bfloat16), (200, 128, torch.float16), (256, 128, torch.bfloat16),
                                       (300, 256, torch.bfloat16), (130, 128, torch.float32), (200, 100, torch.bfloat16)])
def test_single_round_on_either_side_of_its_stream_counts(L, D, dtype, variant):
    """8, 16 and 32 slices a lane, at the stream counts where the choice of the kernel changes (up to a workgroup per
    compute unit, half of that, two per unit), with nothing and with much behind the reference chunk."""
    S = 2
    for H, behind in [(128, 0), (136, 0), (256, L - 1), (264, 0), (264, L - 1), (512, 1)]:
        say("append choice", L, D, dtype, "variant", variant, "streams", H, "behind", behind)
        T = S + 2 * L + behind
        Kh, Vh = gen(1, H, T, D, dtype, seed=L + H)
        cache = lagkv.Cache(1, H, D, T, S, L, 0.25, dtype=dtype, variant=variant)
        first = S + 2 * L - 1
        cache.append_and_compress(Kh[:, :, :first], Vh[:, :, :first])
        assert cache.n_static == S
        cache.append_and_compress(Kh[:, :, first:], Vh[:, :, first:])
        torch.cuda.synchronize()
        few = [0, H // 2, H - 1]
        sub = lagkv.Cache(1, 3, D, T, S, L, 0.25, dtype=dtype, variant=variant)
        sub.K, sub.V, sub.pos = (x[:, few].contiguous() for x in (cache.K, cache.V, cache.pos))
        sub.c = lagkv.CacheT(0, 0, None, T, cache.n_static, cache.n_tail, cache.n_seen)
        oracle_history_check(sub, Kh[:, few], Vh[:, few], S, L, 0.25, VARIANT_NAME[variant])


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("D,dtype,L", [(128, torch.bfloat16, 128), (128, torch.bfloat16, 300), (100, torch.float16, 50)])
def test_an_append_captured_and_replayed(D, dtype, L, variant):
    """The kernels of two calls - rows that complete nothing, then the row that completes a chunk - replayed on the same
    buffers three times, the cache put back and eager work done in between."""
    S, T = 5, 5 + 2 * L
    Kh, Vh = gen(2, 4, T, D, dtype, seed=L + D)
    first = T - 4

    def start():
        cache = lagkv.Cache(2, 4, D, T, S, L, 0.25, dtype=dtype, variant=variant)
        cache.append_and_compress(Kh[:, :, :first].contiguous(), Vh[:, :, :first].contiguous())
        return cache

    parts = [tuple(x[:, :, a:b].contiguous() for x in (Kh, Vh)) for a, b in ((first, T - 1), (T - 1, T))]
    eager, cache = start(), start()
    for part in parts:
        eager.append_and_compress(*part)
    held = [x.clone() for x in (cache.K, cache.V, cache.pos)]
    counters = (cache.c.n_static, cache.c.n_tail, cache.c.n_seen)

    def put_back():
        for x, y in zip((cache.K, cache.V, cache.pos), held):
            x.copy_(y)
        cache.c.n_static, cache.c.n_tail, cache.c.n_seen = counters

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for part in parts:
            cache.append_and_compress(*part)
    torch.cuda.current_stream().wait_stream(side)
    put_back()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for part in parts:
            cache.append_and_compress(*part)
    after = (cache.c.n_static, cache.c.n_tail, cache.c.n_seen)
    for rep in range(3):
        put_back()
        _ = (cache.K.float().sum() + rep).item()
        g.replay()
        torch.cuda.synchronize()
        say("append graph replay", D, L, "variant", variant, rep)
        cache.c.n_static, cache.c.n_tail, cache.c.n_seen = after
        assert all(torch.equal(x, y) for x, y in zip(cache.view(), eager.view()))
    oracle_history_check(cache, Kh, Vh, S, L, 0.25, VARIANT_NAME[variant])
