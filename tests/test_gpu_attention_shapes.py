"""Block shapes of the 64-wide bf16 attention on the GPU: batches on both
sides of the dispatch's lines, against the oracle on sampled heads."""
import numpy as np
import pytest

import oracle as O
from paper_2510_01565_amd import dit, synth
from harness import BF16_TOL, normwise_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grids,n_txt,heads", [
    ([(16, 24)], [0], 256),            # 768 units of 128 queries: 128-query blocks
    ([(16, 24)], [1], 200),            # 800 units, an odd key: 400 256-query blocks of 385 keys
    ([(23, 17)], [0], 270),            # 1080 units, 540 256-query blocks: 128-query blocks again
    ([(16, 24), (5, 5)], [0, 3], 220), # mixed lengths: 128-query blocks
])
def test_attention_d64_dispatch(grids, n_txt, heads):
    import torch
    d, lens = 64, [gh * gw + nt for (gh, gw), nt in zip(grids, n_txt)]
    T = sum(lens)
    q, k, v = (synth.normal(31, n, (T, heads, d), bf16=True) for n in "qkv")
    b = dit.Batch([g[0] for g in grids], [g[1] for g in grids], n_txt)
    wsb = dit.attention_workspace_size(b, heads, d, dit.DIT_BF16)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    o = torch.full((T, heads, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    dit.dit_attention(b, heads, d, dit.DIT_BF16, *(to_dev(x, torch.bfloat16) for x in (q, k, v)), o, ws, wsb)
    torch.cuda.synchronize()
    got = o.float().cpu().numpy()
    assert np.isfinite(got).all()
    hs = [0, 1, heads // 2, heads - 2, heads - 1]
    off = 0
    for L in lens:
        sl = slice(off, off + L)
        ref = O.attention(*(x[sl][:, hs].astype(np.float64) for x in (q, k, v)))
        assert normwise_err(got[sl][:, hs], ref) < BF16_TOL
        off += L


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("gain", [1.0, 16.0])
@pytest.mark.parametrize("grids,n_txt,heads", [
    ([(31, 41)], [0], 3),                  # 1271 keys: 20 tiles, 10 for each key group, the last one ragged
    ([(32, 42)], [0], 2),                  # 1344: 21 tiles, 11 and 10
    ([(36, 36), (1, 1), (8, 16)], [3, 0, 1], 2),  # 21 tiles, one tile (no second group), 3 tiles
])
def test_attention_key_groups(grids, n_txt, heads, d, gain):
    """Few long query tiles: two wave groups share a block's keys; logits up to hundreds put their maxima
    far apart.  Every row against the oracle, and the same bits on a second call."""
    import torch
    lens = [gh * gw + nt for (gh, gw), nt in zip(grids, n_txt)]
    T = sum(lens)
    qb, kb = (torch.from_numpy((synth.normal(32, n, (T, heads, d)) * np.float32(gain ** 0.5))).to(torch.bfloat16) for n in "qk")
    v = synth.normal(32, "v", (T, heads, d), bf16=True)
    b = dit.Batch([g[0] for g in grids], [g[1] for g in grids], n_txt)
    wsb = dit.attention_workspace_size(b, heads, d, dit.DIT_BF16)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    outs = []
    for _ in range(2):
        o = torch.full((T, heads, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        dit.dit_attention(b, heads, d, dit.DIT_BF16, qb.cuda(), kb.cuda(), to_dev(v, torch.bfloat16), o, ws, wsb)
        torch.cuda.synchronize()
        outs.append(o)
    assert torch.equal(outs[0], outs[1])
    got, off = outs[0].float().cpu().numpy(), 0
    q64, k64 = qb.float().numpy().astype(np.float64), kb.float().numpy().astype(np.float64)
    for L in lens:
        sl = slice(off, off + L)
        assert normwise_err(got[sl], O.attention(q64[sl], k64[sl], v[sl].astype(np.float64))) < BF16_TOL
        off += L


@pytest.mark.parametrize("grids,n_txt,heads,shared", [
    ([(92, 92)], [0], 24, True),                          # 34 tiles x 24 heads: 3 rounds and 48 tiles in 256 runs
    ([(92, 92), (20, 25), (1, 1)], [7, 0, 0], 24, True),  # mixed lengths: whole short tiles inside runs
    ([(128, 128)], [512], 6, True),                       # one round, runs shorter than a tile
    ([(64, 64)], [512], 24, False),                       # whole rounds only
])
def test_attention_evenly_shared_keys(grids, n_txt, heads, shared):
    """Sampled rows and heads against the oracle (the rows at both ends of every tile among them), the same
    bits on a second call, and the plan of a workspace without room for the runs' parts."""
    import torch
    d, lens = 128, [gh * gw + nt for (gh, gw), nt in zip(grids, n_txt)]
    T, Tp = sum(lens), sum((L + 63) // 64 * 64 for L in lens)
    gen = torch.Generator(device="cuda").manual_seed(33)
    q, k, v = (torch.randn((T, heads, d), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    b = dit.Batch([g[0] for g in grids], [g[1] for g in grids], n_txt)
    wsb = dit.attention_workspace_size(b, heads, d, dit.DIT_BF16)
    big = (heads * d * Tp * 2 + 255) // 256 * 256 + (66 << 20)
    outs = []
    for n in (big, big, wsb):
        ws = torch.full((n,), 255, dtype=torch.uint8, device="cuda")  # stale parts are NaN
        o = torch.full((T, heads, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        dit.dit_attention(b, heads, d, dit.DIT_BF16, q, k, v, o, ws, n)
        torch.cuda.synchronize()
        outs.append(o)
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(outs[0], outs[2]) != shared
    assert torch.isfinite(outs[0]).all()
    # every element, against the plan without shared keys: two roundings of P to bf16 and one of O apart
    diff = (outs[0].float() - outs[2].float()).norm() / outs[2].float().norm()
    assert diff < 2 ** -7, diff
    rng, off = np.random.default_rng(33), 0
    for L in lens:
        rows = np.unique(np.concatenate([np.arange(0, L, 256), np.arange(255, L, 256), [L - 1],
                                         rng.integers(0, L, min(L, 40))]))
        sl = slice(off, off + L)
        for h in (0, heads // 2, heads - 1):
            x = [t[sl, h:h + 1].float().cpu().numpy().astype(np.float64) for t in (q, k, v)]
            ref = O.attention(*x, rows=rows)
            assert normwise_err(outs[0][sl, h:h + 1].float().cpu().numpy()[rows], ref) < BF16_TOL
        off += L
