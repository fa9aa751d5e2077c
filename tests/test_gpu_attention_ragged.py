"""Attention over batches of mixed lengths: the split of a head over workgroups
follows the pages there are, so heads of one call have different chunk counts.
Every length is checked against the same sequence attended alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv,B,P,d,dtype,factors,longest,lens", [
    (8, 1, 64, 128, "bf16", "bf16", 33 * 64, [[32 * 64], [31 * 64 + 5], [33 * 64]]),
    (8, 1, 64, 128, "bf16", "int4", 33 * 64, [[32 * 64]]),
    (4, 2, 64, 128, "bf16", "bf16", 33 * 64, [[32 * 64, 70], [64, 31 * 64], [2000, 2001]]),
    (4, 1, 16, 96, "f32", "f32", 65 * 16, [[64 * 16], [1]])])
def test_workspace_for_a_longer_length_serves_shorter_ones(Hkv, B, P, d, dtype, factors, longest, lens, monkeypatch):
    """A shorter call may split its heads further than the longest and so ask for more
    partial states; it takes a plan that fits the workspace it is given."""
    import torch
    import paper_2608_23843_amd as pk
    r, G = 8, 2
    g = torch.Generator(device="cuda").manual_seed(longest)
    cache = pk.PuzzleKVCache(1, B, Hkv, Hkv * G, d, P, -(-longest // P), r, P, 2 * P, dtype, factors)
    k, v = (torch.randn(B, Hkv, longest, d, generator=g, device="cuda").to(cache.qdtype) for _ in range(2))
    q = torch.randn(B, Hkv * G, d, generator=g, device="cuda").to(cache.qdtype)
    ws = cache.workspace(pk.PKV_OP_ATTENTION, longest)
    tol = 5e-4 if factors == "int4" else 1e-5   # the order of the fp32 sums
    for n in lens:
        cache.prefill(0, k, v, n, default_rank=(r, r))
        ro, rl = cache.attention(0, q, n)
        with monkeypatch.context() as m:
            m.setattr(torch, "zeros", None)   # the binding makes no workspace of its own
            o, l = cache.attention(0, q, n, workspace=ws)
        assert (o - ro).norm() <= tol * ro.norm() and (l - rl).abs().max() <= tol * float(rl.abs().max())
        assert cache.device_status() == 0


@pytest.mark.parametrize("Hkv,G,P,d,dtype,factors,lens", [
    (1, 8, 64, 128, "bf16", "bf16", [20011, 1, 0, 4097, 64, 9000]),                 # many chunks against one
    (8, 4, 64, 128, "bf16", "bf16", [6001] + [65 + 97 * i for i in range(24)]),      # more heads than CUs would hold
    (2, 2, 32, 64, "bf16", "bf16", [3000, 2990, 2999, 31]),                          # counts that nearly agree
    (4, 1, 16, 128, "bf16", "bf16", [2049, 17, 2048]),
    (8, 8, 64, 128, "bf16", "int4", [5000, 130, 2600]),
    (2, 16, 32, 96, "f32", "f32", [1500, 33, 700, 0]),
    (1, 2, 64, 128, "bf16", "bf16", [700 - i for i in range(200)]),                  # a large batch
    (1, 2, 64, 128, "bf16", "bf16", [640, 64] + [640] * 198)])               # two chunks per sequence but one
def test_mixed_lengths_match_single_sequences(Hkv, G, P, d, dtype, factors, lens):
    import torch
    import paper_2608_23843_amd as pk
    B, S, W, r = len(lens), P, 2 * P, min(P, 16)
    T = max(lens)
    g = torch.Generator(device="cuda").manual_seed(B + T)
    cache = pk.PuzzleKVCache(1, B, Hkv, Hkv * G, d, P, -(-T // P), r, S, W, dtype, factors)
    k, v = (torch.randn(B, Hkv, T, d, generator=g, device="cuda").to(cache.qdtype) for _ in range(2))
    cache.prefill(0, k, v, lens, default_rank=(r, r))
    q = torch.randn(B, Hkv * G, d, generator=g, device="cuda").to(cache.qdtype)
    ws = cache.workspace(pk.PKV_OP_ATTENTION, T)
    outs = [tuple(x.clone() for x in cache.attention(0, q, lens, workspace=ws)) for _ in range(2)]
    na = torch.empty_like(outs[0][0]), torch.empty_like(outs[0][1])
    outs.append(cache.attention_noalloc(0, q, lens, *na) if B * Hkv <= 2048 else outs[0])
    assert cache.device_status() == 0
    # alone: every other sequence empty
    tol = 5e-4 if factors == "int4" else 1e-5   # the order of the fp32 sums (INT4: of fp16 hi/lo products)
    for b in {0, 1, B // 2, B - 1}:
        if lens[b] == 0:
            for o, l in outs:
                assert torch.all(o[b] == 0) and torch.all(torch.isneginf(l[b]))
            continue
        ro, rl = cache.attention(0, q, [n if i == b else 0 for i, n in enumerate(lens)], workspace=ws)
        for o, l in outs:
            assert (o[b] - ro[b]).norm() <= tol * ro[b].norm(), b
            assert (l[b] - rl[b]).abs().max() <= tol * max(1.0, float(rl[b].abs().max())), b
