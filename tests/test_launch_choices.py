"""GPU: the one-shot pass under its own launch choices (nothing hinted), at the sizes where the split of
the work can go wrong: one chunk per segment and several in each kernel, sink and window rows in one share and in
many, shares of one row, no sink, a window of one lag exactly."""
import pytest
import torch

from paper_2504_04704_amd import lagkv
from tests import parity_util as PU
from tests.test_gpu_parity import VARIANT_NAME, gen, oracle_history_check, run_and_check, say

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


# Rows that are not whole 16-byte slices, on 4-byte aligned addresses: the chunk-at-a-time kernel, against
# the three-kernel path on the same bytes.  Row sizes at both ends of its range and around whole slices.
PARTIAL_ROWS = [(100, torch.bfloat16), (50, torch.float16), (10, torch.bfloat16), (34, torch.bfloat16), (66, torch.float16),
                (5, torch.float32), (33, torch.float32), (126, torch.float32), (254, torch.bfloat16), (130, torch.float16)]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("D,dtype", PARTIAL_ROWS)
def test_rows_of_partial_slices_against_the_staged_path(D, dtype, variant):
    say("partial slices", D, dtype, "variant", variant)
    staged = lagkv.launch_hint(lagkv.PATH_STAGED)
    for n, (S, L, r) in enumerate([(3, 37, 0.3), (16, 128, 0.25), (0, 129, 0.5), (1, 256, 0.125), (2, 300, 0.2)]):
        T = S + 4 * L + 11
        K, V = gen(2, 3, T, D, dtype, seed=D + n)
        if n % 2:  # the layout of attention kernels, the base moved by two tokens
            K, V = (torch.cat([x[:, :, :2], x], 2).transpose(1, 2).contiguous()[:, 2:].transpose(1, 2) for x in (K, V))
        out, _ = run_and_check(K, V, S, L, r, variant=variant, streams=[(0, 0), (1, 2)])
        ref = lagkv.compress(K, V, S, L, r, variant=variant, want_scores=True, launch=staged)
        torch.cuda.synchronize()
        # two fp32 summation orders of the same sums: a few ulp of a standard deviation of order one (the bound of
        # 2e-6 is the derivation of the scoring kernels' own)
        assert torch.allclose(out.scores, ref.scores, rtol=4e-6, atol=0)
        assert torch.equal(lagkv.score(K, V, S, L, r, variant=variant), out.scores)


def test_row_strides_that_are_not_whole_slices():
    """Rows of 128 bytes in a tensor whose row stride is 132 bytes: no longer read element by element."""
    K, V = gen(1, 2, 700, 66, torch.bfloat16, seed=3)
    K, V = K[..., :64], V[..., :64]
    assert lagkv.workspace_bytes(lagkv.params_for(K, 16, 100, 0.25), 700) > 0
    run_and_check(K, V, 16, 100, 0.25)
    # equal tokens across the edge of the kept set, both counting ranges
    for L in (60, 128, 250):
        K2, V2 = K.clone(), V.clone()
        K2[:, :, 16:16 + 2 * L] = K[:, :, 16:17]
        V2[:, :, 16:16 + 2 * L] = V[:, :, 16:17]
        K2[:, :, 16 + 2 * L:16 + 2 * L + 5] = K[:, :, 300:305]
        run_and_check(K2[..., :62], V2[..., :62], 16, L, 0.3)


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL])
@pytest.mark.parametrize("D,L", [(50, 64), (33, 200), (50, 300), (126, 128), (48, 100)])
def test_channel_offsets_far_above_the_ranges(D, L, variant):
    """fp32 channels at a million times their range: x - min is exact there (the two are within a factor of two of
    each other), so the scores are as good as anywhere, and the bar against the oracle is the same 1e-5."""
    say("channel offsets", D, L, "variant", variant)
    S, T = 3, 3 + 6 * L + 11
    g = torch.Generator(device="cuda").manual_seed(D + L)
    K, V = (4e6 * (1 + torch.rand((1, 2, 1, D), generator=g, device="cuda"))
            + 4 * torch.randn((1, 2, T, D), generator=g, device="cuda") for _ in range(2))
    run_and_check(K, V, S, L, 0.25, variant=variant)
    cache = lagkv.Cache(1, 2, D, T, S, L, 0.25, dtype=torch.float32, variant=variant)
    for a, b in [(0, S + 2 * L - 1), (S + 2 * L - 1, S + 2 * L), (S + 2 * L, S + 3 * L)]:
        cache.append_and_compress(K[:, :, a:b], V[:, :, a:b])
    torch.cuda.synchronize()
    oracle_history_check(cache, K[:, :, :b], V[:, :, :b], S, L, 0.25, VARIANT_NAME[variant])


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL])
@pytest.mark.parametrize("B,H,n,m,L,S", [(2, 128, 2, 0, 128, 16), (2, 128, 5, 127, 128, 0), (1, 200, 2, 100, 128, 700), (1, 224, 3, 255, 256, 1),
                                         (2, 256, 2, 3, 512, 16), (1, 700, 2, 77, 128, 3), (1, 96, 9, 20, 128, 5)])
def test_sink_and_window_rows_copied_in_line(B, H, n, m, L, S, variant):
    """Streams that fill the compute units, or nearly: the resident kernel's scoring workgroups copy these rows themselves
    (the last case, with room, and the positions of every stream, beside it)."""
    say("edge rows in line", B, H, n, m, L, S, "variant", variant)
    T = S + n * L + m
    K, V = gen(B, H, T, 128, torch.bfloat16, seed=H + n)
    out, _ = run_and_check(K, V, S, L, 0.25, variant=variant, streams=[(0, 0), (B - 1, H // 2), (B - 1, H - 1)])
    PU.check_index_invariants(out.idx, T, S, L, L // 4, n - 1)
    rows = out.idx.long().unsqueeze(-1).expand(-1, -1, -1, 128)
    assert torch.equal(out.K, K.gather(2, rows)) and torch.equal(out.V, V.gather(2, rows))


def on_odd_addresses(x, pad, shift):
    """The same values with `pad` more channels from row to row, `shift` channels into the allocation."""
    B, H, T, D = x.shape
    flat = torch.full((B * H * T * (D + pad) + shift,), 7, dtype=x.dtype, device=x.device)
    view = flat[shift:].as_strided((B, H, T, D), (H * T * (D + pad), T * (D + pad), D + pad, 1), shift)
    view.copy_(x)
    return view


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("D,dtype", [(32, torch.bfloat16), (64, torch.float16), (32, torch.float32), (128, torch.bfloat16), (256, torch.bfloat16)])
def test_whole_rows_on_four_byte_addresses(D, dtype, variant):
    """Rows of 64, 128, 256 and 512 bytes that start on any multiple of 4: one-shot and as the new rows of a cache."""
    step = 4 // dtype.itemsize
    for L, pad, shift in [(64, step, 0), (128, 3 * step, step), (130, 2 * step, 3 * step), (300, step, 2 * step)]:
        say("four-byte addresses", D, dtype, "variant", variant, "L", L, "pad", pad, "shift", shift)
        S, T = 5, 5 + 4 * L + 9
        K0, V0 = gen(1, 3, T, D, dtype, seed=D + L)
        K, V = on_odd_addresses(K0, pad, shift), on_odd_addresses(V0, pad, shift)
        assert K.data_ptr() % 16 == 4 * (shift // step) and torch.equal(K, K0)
        out, _ = run_and_check(K, V, S, L, 0.3, variant=variant)
        want = lagkv.compress(K0, V0, S, L, 0.3, variant=variant)
        cache = lagkv.Cache(1, 3, D, T, S, L, 0.3, dtype=dtype, variant=variant)
        for a, b in [(0, S + 2 * L - 1), (S + 2 * L - 1, S + 2 * L), (S + 2 * L, T - L), (T - L, T)]:
            cache.append_and_compress(K[:, :, a:b], V[:, :, a:b])
        torch.cuda.synchronize()
        oracle_history_check(cache, K, V, S, L, 0.3, VARIANT_NAME[variant])
        assert torch.equal(out.K, want.K) and torch.equal(out.V, want.V) and torch.equal(out.idx, want.idx)


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("D,dtype,pad,shift", [(128, torch.bfloat16, 0, 2), (128, torch.bfloat16, 8, 6), (96, torch.float16, 0, 4), (64, torch.float32, 4, 3)])
def test_whole_strides_on_a_four_byte_base_need_no_workspace(D, dtype, pad, shift, variant):
    """lagkv_workspace_bytes, which sees no addresses, answers 0: the pass, and a cache's rows up to and over the one that
    completes a chunk, take tensors (the cache's own among them) that start 4, 8 or 12 bytes into a slice."""
    say("four-byte base", D, dtype, pad, shift, "variant", variant)
    S, L = 5, 100
    T = S + 4 * L + 9
    K, V = (on_odd_addresses(x, pad, shift) for x in gen(2, 3, T, D, dtype, seed=D + shift))
    assert K.data_ptr() % 16 != 0 and lagkv.workspace_bytes(lagkv.params_for(K, S, L, 0.3, variant), T) == 0
    run_and_check(K, V, S, L, 0.3, variant=variant)
    for odd_cache in (False, True):
        cache = lagkv.Cache(2, 3, D, T, S, L, 0.3, dtype=dtype, variant=variant)
        if odd_cache:
            cache.K, cache.V = (on_odd_addresses(x, 0, shift) for x in (cache.K, cache.V))
            cache.c.K, cache.c.V = cache.K.data_ptr(), cache.V.data_ptr()
        for a, b in [(0, S + 2 * L - 1), (S + 2 * L - 1, S + 2 * L), (S + 2 * L, S + 3 * L - 1), (S + 3 * L - 1, S + 4 * L - 2)]:
            cache.append_and_compress(K[:, :, a:b], V[:, :, a:b])
        torch.cuda.synchronize()
        oracle_history_check(cache, K[:, :, :b], V[:, :, :b], S, L, 0.3, VARIANT_NAME[variant])


# streams, scored chunks, D, dtype, L: several chunks per workgroup of the chunk kernel (512 places up to 8 slices a
# lane, else 256), in each range of its selection, on partial and on whole rows.  By Eq. 16 the calls are its own; by the
# others most are the ring kernel's
LONG_RUNS = [
    (64, 21, 100, torch.bfloat16, 128), (40, 40, 100, torch.bfloat16, 64), (64, 13, 100, torch.bfloat16, 200), (64, 9, 100, torch.float16, 300),
    (300, 3, 126, torch.float32, 128), (70, 19, 34, torch.bfloat16, 512), (7, 160, 33, torch.float32, 60),
    (72, 12, 80, torch.bfloat16, 100), (90, 5, 64, torch.bfloat16, 500), (1, 1000, 96, torch.float16, 40), (120, 4, 96, torch.float32, 128),
]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("streams,n_s,D,dtype,L", LONG_RUNS)
def test_several_chunks_per_workgroup(streams, n_s, D, dtype, L, variant):
    """A workgroup that walks a run of chunks: the statistics handed from one to the next, rows loaded behind the stores
    of the one before, the chunk's own statistics (Eq. 14-15), scores alone."""
    whole = D * dtype.itemsize % 16 == 0
    if whole and variant == lagkv.SCORE_L2:  # half the places at most go to it: a scores-only call takes more
        n_s = max(1, 120 // streams)
    S, T = 3, 3 + (n_s + 1) * L + 5
    say("long runs", streams, n_s, D, dtype, L, "variant", variant)
    K, V = gen(1, streams, T, D, dtype, seed=streams + L)
    p = lagkv.params_for(K, S, L, 0.3, variant)
    assert lagkv.kernel_for(p, T) in (("chunk_pass_kernel",) if variant == lagkv.SCORE_L2 or (D, L) == (100, 300) else ("chunk_pass_kernel", "ring_pass_kernel"))
    assert n_s * streams > 256 * (2 if L * D * dtype.itemsize <= 32 * 1024 else 1) or (whole and variant == lagkv.SCORE_L2)
    out, _ = run_and_check(K, V, S, L, 0.3, variant=variant, streams=[(0, s) for s in sorted({0, streams // 2, streams - 1})])
    PU.check_index_invariants(out.idx, T, S, L, out.plan.k, n_s)
    rows = out.idx.long().unsqueeze(-1).expand(-1, -1, -1, D)
    assert torch.equal(out.K, K.gather(2, rows)) and torch.equal(out.V, V.gather(2, rows))
    assert torch.equal(lagkv.score(K, V, S, L, 0.3, variant=variant), out.scores)
    if streams * n_s < 1500:
        ref = lagkv.score(K, V, S, L, 0.3, variant=variant, launch=lagkv.launch_hint(lagkv.PATH_STAGED))
        assert torch.allclose(out.scores, ref, rtol=4e-6, atol=0)     # (as for partial slices above)


# D, dtype, rows of a step of the chunk kernel: whole and partial rows of 64, 128, 256 and 512 bytes
STEPS = [(16, torch.float32, 64), (9, torch.float32, 64), (64, torch.bfloat16, 32), (50, torch.float16, 32), (128, torch.float16, 16),
         (100, torch.bfloat16, 16), (128, torch.float32, 8), (250, torch.bfloat16, 8)]


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("D,dtype,R", STEPS)
def test_chunks_of_one_two_and_three_steps(D, dtype, R, variant):
    """A lag of one row, a row short of a step, one step, one row more, two steps, one row more: the kernel for up to two
    slices a lane and the one for up to eight, one chunk a workgroup and several."""
    for streams, n_s in ((3, 3), (280, 4)):
        for L in (1, R - 1, R, R + 1, 2 * R, 2 * R + 1):
            S, r = (3, 0.3) if L > 3 else (0, 1.0)
            T = S + (n_s + 1) * L + L // 2
            say("steps", streams, D, dtype, L, "variant", variant)
            K, V = gen(1, streams, T, D, dtype, seed=L)
            out, _ = run_and_check(K, V, S, L, r, variant=variant, streams=[(0, s) for s in (0, 1, streams - 1)])
            PU.check_index_invariants(out.idx, T, S, L, out.plan.k, n_s)
            rows = out.idx.long().unsqueeze(-1).expand(-1, -1, -1, D)
            assert torch.equal(out.K, K.gather(2, rows)) and torch.equal(out.V, V.gather(2, rows))
            assert torch.equal(lagkv.score(K, V, S, L, r, variant=variant), out.scores)


@pytest.mark.parametrize("variant", [lagkv.SCORE_LAG, lagkv.SCORE_LOCAL, lagkv.SCORE_L2])
@pytest.mark.parametrize("D,dtype,L", [(100, torch.bfloat16, 60), (100, torch.float16, 128), (33, torch.float32, 250), (66, torch.bfloat16, 400), (80, torch.bfloat16, 300)])
def test_infinities_and_nan_stay_in_their_streams(D, dtype, L, variant):
    """Scores of such rows are unspecified, but every chunk keeps k rows of its own, in order and bit for bit, and the
    streams beside them are what they are without: one-shot and in a cache whose chunk completes."""
    S, n = 5, 4
    T = S + n * L + 7
    say("inf and nan", D, dtype, L, "variant", variant)
    K, V = gen(1, 6, T, D, dtype, seed=D + L)
    want = lagkv.compress(K, V, S, L, 0.3, variant=variant, want_scores=True)
    bad = torch.randperm(T, generator=torch.Generator().manual_seed(L))[: T // 3].cuda()
    K[:, 1, bad, 3], V[:, 2, bad, D - 1] = float("nan"), float("inf")
    K[:, 3], V[:, 3] = float("nan"), -float("inf")
    K[:, 4, ::2, 0], K[:, 4, 1::2, D - 1] = float("inf"), -float("inf")
    out = lagkv.compress(K, V, S, L, 0.3, variant=variant, want_scores=True)
    cache = lagkv.Cache(1, 6, D, T, S, L, 0.3, dtype=dtype, variant=variant)
    for a, b in [(0, S + 2 * L - 2), (S + 2 * L - 2, S + 2 * L + 1), (S + 2 * L + 1, S + 3 * L + 1), (S + 3 * L + 1, T)]:
        cache.append_and_compress(K[:, :, a:b], V[:, :, a:b])
    torch.cuda.synchronize()
    bits = {2: torch.int16, 4: torch.int32}[dtype.itemsize]
    ck, cv, cpos = cache.view()
    for gk, gv, idx in ((out.K, out.V, out.idx), (ck.contiguous(), cv.contiguous(), cpos.contiguous())):
        PU.check_index_invariants(idx, T, S, L, out.plan.k, n - 1)
        rows = idx.long().unsqueeze(-1).expand(-1, -1, -1, D)
        assert torch.equal(gk.view(bits), K.gather(2, rows).view(bits)) and torch.equal(gv.view(bits), V.gather(2, rows).view(bits))
    for s in (0, 5):
        assert torch.equal(out.scores[:, s], want.scores[:, s]) and torch.equal(out.idx[:, s], want.idx[:, s])
        assert torch.equal(cpos[:, s], want.idx[:, s])


@pytest.mark.parametrize("D,dtype,L", [(100, torch.bfloat16, 128), (80, torch.bfloat16, 100), (66, torch.float16, 300)])
def test_chunk_kernel_in_a_captured_graph(D, dtype, L):
    """(The chunk kernel for the last shape, the ring kernel for the others) ... and replayed three times, with eager work between, on other bytes in the same buffers too."""
    S, T = 16, 16 + 5 * L + 17
    K, V = gen(2, 4, T, D, dtype, seed=404)
    p = lagkv.params_for(K, S, L, 0.25)
    assert lagkv.kernel_for(p, T) == ("chunk_pass_kernel" if L == 300 else "ring_pass_kernel")
    want = lagkv.compress(K, V, S, L, 0.25, want_scores=True)
    out = [torch.zeros_like(x) for x in (want.K, want.V, want.idx, want.scores)]
    ws = torch.empty(max(lagkv.workspace_bytes(p, T), 16), dtype=torch.uint8, device="cuda")

    def call():
        lagkv.compress(K, V, S, L, 0.25, out=(out[0], out[1]), idx_out=out[2], scores_out=out[3], ws=ws)

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
            for x, y in zip((K, V), gen(2, 4, T, D, dtype, seed=405)):
                x.copy_(y)
            want = lagkv.compress(K, V, S, L, 0.25, want_scores=True)
        for x in out:
            x.zero_()
        _ = (K.float().sum() + rep).item()
        g.replay()
        torch.cuda.synchronize()
        say("chunk graph replay", D, L, rep)
        assert all(torch.equal(x, y) for x, y in zip(out, (want.K, want.V, want.idx, want.scores)))
