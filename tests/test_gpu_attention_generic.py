"""Attention over fp32 storage and over geometries the bf16 matrix-core kernel
does not take (other head sizes, ranks above 32, mixed storage): the page loop
in fp32 products, against the oracle over the same stored values."""
import numpy as np
import pytest

import oracle
from helpers import storage_round

pytestmark = pytest.mark.gpu

# fp32 products and sums over up to 600 keys and 64 ranks: a few hundred
# roundings of 2^-24 that average out, 1e-5 of the output's norm
REL = 1e-5


@pytest.mark.parametrize("dense,factors,d,P,G,rk,rv", [
    ("f32", "f32", 32, 16, 1, 1, 16), ("f32", "f32", 64, 64, 16, 64, 33), ("f32", "f32", 96, 32, 5, 17, 3),
    ("f32", "f32", 256, 64, 16, 5, 48), ("f32", "bf16", 160, 32, 4, 16, 32), ("bf16", "f32", 128, 16, 8, 9, 7),
    ("bf16", "bf16", 192, 64, 3, 33, 64), ("bf16", "bf16", 32, 32, 2, 8, 8)])
@pytest.mark.parametrize("pages", [1, 9, 41])
def test_generic_attention(dense, factors, d, P, G, rk, rv, pages):
    import torch
    import paper_2608_23843_amd as pk
    if pages == 41 and P == 64:
        pages = 21
    rng = np.random.default_rng(d * P + pages)
    Hkv, S, W = 2, P, P + 3
    lens = [P * (pages - 1) + 1 + int(rng.integers(0, P - 1)), 0, max(1, P * pages // 3)]   # the last page partial
    B = len(lens)
    cache = pk.PuzzleKVCache(1, B, Hkv, Hkv * G, d, P, pages + 1, min(P, max(rk, rv)), S, W, dense, factors)
    # rows nobody has written hold NaN bits
    cache.dense_pool.fill_(0xff)
    cache.factor_pool.fill_(0xff)
    rk, rv = min(rk, P), min(rv, P)
    heads = {}
    for b, T in enumerate(lens):
        plan = oracle.plan_pages(T, P, S, W)
        for h in range(Hkv):
            stored = []
            for j, kind in enumerate(plan):
                if kind == oracle.FACTOR:
                    f = [storage_round(rng.standard_normal(s) * w, factors) for s, w in
                         (((P, rk), P ** -0.5), ((rk, d), 2.0), ((P, rv), P ** -0.5), ((rv, d), 2.0))]
                    src = torch.from_numpy(np.concatenate([x.ravel() for x in f])).to("cuda", cache.fdtype)
                    cache.import_pages(0, [b], [h], [j], [pk.PKV_FACTOR], [rk], [rv], src, [0])
                    stored.append(("factor", *[x.astype(np.float64) for x in f]))
                else:
                    rows = min(P, T - j * P)
                    kv = storage_round(rng.standard_normal((2, rows, d)), dense)
                    stored.append(("dense", *kv.astype(np.float64)))
            heads[b, h] = stored
    # the dense pages arrive token by token, so that the rest of a partial page keeps its NaN bits
    for t in range(max(lens)):
        kv = np.zeros((2, B, Hkv, d), dtype=np.float32)
        pos = [-1] * B
        for b, T in enumerate(lens):
            if t < T and heads[b, 0][t // P][0] == "dense":
                pos[b] = t
                for h in range(Hkv):
                    kv[:, b, h] = [x[t % P] for x in heads[b, h][t // P][1:]]
        if max(pos) >= 0:
            k, v = torch.from_numpy(kv).to("cuda", cache.qdtype)
            cache.append(0, k.contiguous(), v.contiguous(), pos)
    assert cache.device_status() == 0
    q = storage_round(rng.standard_normal((B, Hkv * G, d)) * 1.5, dense)
    qt = torch.from_numpy(q).to("cuda", cache.qdtype).contiguous()
    ws = cache.workspace(pk.PKV_OP_ATTENTION, max(lens))
    for _ in range(2):   # the second call finds the workspace as the first left it
        out, lse = cache.attention(0, qt, lens, workspace=ws)
    out, lse = out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    assert cache.device_status() == 0
    for b, T in enumerate(lens):
        if T == 0:
            assert np.all(out[b] == 0) and np.all(np.isneginf(lse[b]))
            continue
        for h in range(Hkv):
            pages_ = [(p[0], *[np.pad(x, ((0, P - len(x)), (0, 0))) for x in p[1:]]) if p[0] == "dense" else p
                      for p in heads[b, h]]
            ro, rl = oracle.attention(oracle.HeadCache(T, P, d, pages_), q[b, h * G:(h + 1) * G].astype(np.float64))
            got = out[b, h * G:(h + 1) * G]
            assert np.linalg.norm(got - ro) <= REL * np.linalg.norm(ro), (b, h)
            assert np.abs(lse[b, h * G:(h + 1) * G] - rl).max() <= REL * max(1.0, np.abs(rl).max())


@pytest.mark.parametrize("dense,d,P", [("f32", 96, 32), ("bf16", 160, 64), ("f32", 32, 16)])
def test_minus_infinity_key_entries(dense, d, P):
    """Keys whose last dims hold -inf where the query is positive score -inf and get no
    weight, also where the head is not a whole number of the kernel's dim tiles."""
    import torch
    import paper_2608_23843_amd as pk
    Hkv, G, T = 2, 3, 5 * P - 7
    g = torch.Generator(device="cuda").manual_seed(d)
    cache = pk.PuzzleKVCache(1, 1, Hkv, Hkv * G, d, P, 5, 4, P, 5 * P, dense, dense)   # every page in the window
    k, v = (torch.randn(1, Hkv, T, d, generator=g, device="cuda").to(cache.qdtype) for _ in range(2))
    q = torch.randn(1, Hkv * G, d, generator=g, device="cuda").to(cache.qdtype)
    q[..., -3] = q[..., -3].abs() + 0.1
    out_at = torch.arange(T, device="cuda") % 3 == 1
    k[:, :, out_at, -3] = -float("inf")
    cache.prefill(0, k, v, [T], default_rank=(1, 1))
    out, lse = cache.attention(0, q, [T])
    assert cache.device_status() == 0
    for h in range(Hkv):
        kk, vv = k[0, h, ~out_at].double(), v[0, h, ~out_at].double()
        s = q[0, h * G:(h + 1) * G].double() @ kk.T.contiguous() / d ** 0.5
        ref = torch.softmax(s, 1) @ vv
        assert (out[0, h * G:(h + 1) * G].double() - ref).norm() <= REL * ref.norm()
        assert (lse[0, h * G:(h + 1) * G].double() - torch.logsumexp(s, 1)).abs().max() <= REL * 10
