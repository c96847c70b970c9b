"""Block shapes of the 64-wide bf16 attention on the GPU: batches on both
sides of the dispatch's lines, against the oracle on sampled heads."""
import numpy as np
import pytest

import oracle as O
from paper_2510_01565_amd import dit, synth, workloads
from harness import BF16_TOL, F32_TOL, normwise_err, to_dev

pytestmark = pytest.mark.gpu

SHARE_BYTES = 66 << 20  # past V^T: leave for plans whose sums depend on the batch


def _vt_bytes(lens, heads, d):
    return (heads * d * sum((L + 63) // 64 * 64 for L in lens) * 2 + 255) // 256 * 256


def _plans(profile):
    """The attention plans of a profiled run."""
    return {k.rsplit("attention_bf16_", 1)[1] for k in profile if k.startswith("detail:attention_bf16_")}


@pytest.mark.parametrize("grids,n_txt,heads,plan", [
    ([(16, 24)], [0], 256, "128"),            # 768 units of 128 queries
    ([(16, 24)], [1], 200, "256"),            # 800 units, an odd key: 400 256-query blocks of 385 keys
    ([(23, 17)], [0], 270, "128"),            # 1080 units, 540 256-query blocks: the last round nearly empty
    ([(16, 24), (5, 5)], [0, 3], 220, "128"), # mixed lengths, more than 512 256-query blocks
    ([(16, 24), (16, 23)], [1, 0], 120, "256"),  # mixed lengths: 840 units, 480 256-query blocks
])
def test_attention_d64_dispatch(grids, n_txt, heads, plan):
    import torch
    d, lens = 64, [gh * gw + nt for (gh, gw), nt in zip(grids, n_txt)]
    T = sum(lens)
    q, k, v = (synth.normal(31, n, (T, heads, d), bf16=True) for n in "qkv")
    b = dit.Batch([g[0] for g in grids], [g[1] for g in grids], n_txt)
    wsb = dit.attention_workspace_size(b, heads, d, dit.DIT_BF16)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    o = torch.full((T, heads, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    dit.profile_start()
    dit.dit_attention(b, heads, d, dit.DIT_BF16, *(to_dev(x, torch.bfloat16) for x in (q, k, v)), o, ws, wsb)
    torch.cuda.synchronize()
    assert _plans(dit.profile_stop()) == {plan}
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
@pytest.mark.parametrize("grids,n_txt,heads,plan", [
    ([(31, 41)], [0], 3, "128"),                  # 1271 keys, fewer than 20 whole tiles: no groups
    ([(32, 40)], [0], 3, "key_groups"),           # 1280: 20 tiles, 10 for each key group
    ([(31, 42)], [0], 3, "key_groups"),           # 1302: 21 tiles, 11 and 10, the last one ragged
    ([(32, 42)], [0], 2, "key_groups"),           # 1344: 21 tiles, 11 and 10
    ([(36, 36), (1, 1), (8, 16)], [3, 0, 1], 2, "key_groups"),  # 21 tiles, one tile (no second group), 3 tiles
])
def test_attention_key_groups(grids, n_txt, heads, plan, d, gain):
    """Few long query tiles: two wave groups share a block's keys; logits up to hundreds put their maxima
    far apart.  Every row against the oracle, and the same bits on a second call."""
    import torch
    lens = [gh * gw + nt for (gh, gw), nt in zip(grids, n_txt)]
    T = sum(lens)
    qb, kb = (torch.from_numpy((synth.normal(32, n, (T, heads, d)) * np.float32(gain ** 0.5))).to(torch.bfloat16) for n in "qk")
    v = synth.normal(32, "v", (T, heads, d), bf16=True)
    b = dit.Batch([g[0] for g in grids], [g[1] for g in grids], n_txt)
    wsb = _vt_bytes(lens, heads, d) + SHARE_BYTES
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    outs = []
    dit.profile_start()
    for _ in range(2):
        o = torch.full((T, heads, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        dit.dit_attention(b, heads, d, dit.DIT_BF16, qb.cuda(), kb.cuda(), to_dev(v, torch.bfloat16), o, ws, wsb)
        torch.cuda.synchronize()
        outs.append(o)
    assert _plans(dit.profile_stop()) == {plan}
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
    T = sum(lens)
    gen = torch.Generator(device="cuda").manual_seed(33)
    q, k, v = (torch.randn((T, heads, d), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    b = dit.Batch([g[0] for g in grids], [g[1] for g in grids], n_txt)
    wsb = dit.attention_workspace_size(b, heads, d, dit.DIT_BF16)
    big = _vt_bytes(lens, heads, d) + SHARE_BYTES
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


@pytest.mark.parametrize("d", [128, 64])
def test_attention_bits_do_not_depend_on_the_batch(d):
    """At the reported workspace size a request of 1344 keys has the same bits alone (33 query tiles) and packed
    (more than 256), at both ends of the batch."""
    import torch
    heads, grids, n_txt = 3, [(32, 42), (64, 64), (64, 66), (64, 63), (32, 42)], [0, 0, 5, 512, 0]
    lens = [gh * gw + nt for (gh, gw), nt in zip(grids, n_txt)]
    assert sum((L + 127) // 128 for L in lens) * heads > 256
    gen = torch.Generator(device="cuda").manual_seed(34)
    q, k, v = (torch.randn((sum(lens), heads, d), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))

    def run(rs, sl):
        b = dit.Batch([grids[r][0] for r in rs], [grids[r][1] for r in rs], [n_txt[r] for r in rs])
        n = dit.attention_workspace_size(b, heads, d, dit.DIT_BF16)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        x = [t[sl].contiguous() for t in (q, k, v)]
        o = torch.full_like(x[0], float("nan"))
        dit.dit_attention(b, heads, d, dit.DIT_BF16, *x, o, ws, n)
        torch.cuda.synchronize()
        return o

    packed, off = run(range(len(lens)), slice(None)), 0
    assert torch.isfinite(packed).all()
    for r, L in enumerate(lens):
        sl = slice(off, off + L)
        assert torch.equal(run([r], sl), packed[sl]), r
        off += L


@pytest.mark.parametrize("head_dim", [128, 64])
@pytest.mark.parametrize("kind", [0, 1])
def test_batch_invariant_block_keeps_key_groups_out(kind, head_dim):
    """A request of 1344 tokens and few heads: alone its attention would run two key groups per block, packed it
    has more than 256 query tiles.  Batch-invariant blocks give it the same bits in both."""
    import torch
    heads = 4
    m = workloads.ModelShape(hidden=heads * head_dim, heads=heads, head_dim=head_dim, mlp_ratio=1, n_double=1 - kind,
                             n_single=kind, in_channels=64, text_dim=64)
    grids, n_txt = [(36, 36), (64, 64), (60, 64)], [48, 100, 0]
    H, lens = m.hidden, [gh * gw + nt for (gh, gw), nt in zip(grids, n_txt)]
    assert lens[0] == 1344 and sum((L + 127) // 128 for L in lens) * heads > 256
    gen = torch.Generator(device="cuda").manual_seed(35)
    w = dit.Weights([torch.randn(s, generator=gen, device="cuda").mul_(0.05).to(torch.bfloat16)
                     for _, s in dit.weight_manifest(dit.make_config(m))])
    txt = [torch.randn((n, H), generator=gen, device="cuda") for n in n_txt]
    img = [torch.randn((gh * gw, H), generator=gen, device="cuda") for gh, gw in grids]
    cond = torch.randn((len(lens), H), generator=gen, device="cuda")

    def run(rs, flags):
        cfg = dit.make_config(m, flags)
        b = dit.Batch([grids[r][0] for r in rs], [grids[r][1] for r in rs], [n_txt[r] for r in rs])
        n = dit.workspace_size(cfg, b)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        hidden = torch.cat([txt[r] for r in rs] + [img[r] for r in rs])
        dit.profile_start()
        dit.dit_block_forward(cfg, w, kind, 0, b, hidden, cond[rs].contiguous(), ws, n)
        torch.cuda.synchronize()
        return hidden, _plans(dit.profile_stop())

    assert run([0], 0)[1] == {"key_groups"}
    alone, plans = run([0], dit.DIT_FLAG_BATCH_INVARIANT)
    assert plans == {"128"}
    packed, _ = run([0, 1, 2], dit.DIT_FLAG_BATCH_INVARIANT)
    T = sum(n_txt)
    assert torch.isfinite(packed).all()
    assert torch.equal(alone[:n_txt[0]], packed[:n_txt[0]])
    assert torch.equal(alone[n_txt[0]:], packed[T:T + 36 * 36])


@pytest.mark.parametrize("bf16,d,grid,n_txt,heads,cut,plan", [
    (False, 64, (16, 16), 32, 2, [(64, 80), (128, 176), (256, 288)], None),  # first tiles of the waves, the last tile
    (False, 64, (5, 7), 0, 1, [(0, 16), (32, 35)], None),                    # waves of one tile each
    (True, 128, (32, 42), 0, 2, [(704, 768)], "key_groups"),    # the second group's first tile
    (True, 64, (32, 42), 0, 2, [(704, 1344)], "key_groups"),    # all of the second group
    (True, 64, (32, 42), 0, 2, [(0, 704)], "key_groups"),       # all of the first
    (True, 128, (128, 128), 512, 6, [(4000, 16896)], "shared"),  # most runs' whole shares
    (True, 128, (16, 16), 0, 2, [(0, 64), (128, 256)], "128"),  # the first tile of a plain block
])
def test_attention_keys_without_weight(bf16, d, grid, n_txt, heads, cut, plan):
    """Keys whose scores are -inf for every query (a coordinate of -inf against a positive one) have weight zero,
    also where they fill a wave's, a group's or a run's first tiles: the result is attention over the other keys."""
    import torch
    L = grid[0] * grid[1] + n_txt
    dt = torch.bfloat16 if bf16 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(36)
    q, k, v = (torch.randn((L, heads, d), generator=gen, device="cuda").to(dt) for _ in range(3))
    q[..., 0] = 1.0
    keep = torch.ones(L, dtype=torch.bool, device="cuda")
    for a, e in cut:
        k[a:e, :, 0] = float("-inf")
        keep[a:e] = False
    b = dit.Batch([grid[0]], [grid[1]], [n_txt])
    et = dit.DIT_BF16 if bf16 else dit.DIT_F32
    n = _vt_bytes([L], heads, d) + SHARE_BYTES if bf16 else dit.attention_workspace_size(b, heads, d, et)
    ws, o = torch.empty(n, dtype=torch.uint8, device="cuda"), torch.full_like(q, float("nan"))
    dit.profile_start()
    dit.dit_attention(b, heads, d, et, q, k, v, o, ws, n)
    torch.cuda.synchronize()
    plans = _plans(dit.profile_stop())
    assert plans == ({plan} if plan else set())
    rows = np.unique(np.concatenate([np.arange(0, L, 131), [L - 1]]))
    for h in range(heads):
        qh, kh, vh = (x[:, h].double().cpu().numpy() for x in (q, k[keep], v[keep]))
        s = qh[rows] @ kh.T / np.sqrt(d)
        p = np.exp(s - s.max(axis=1, keepdims=True))
        ref = (p / p.sum(axis=1, keepdims=True)) @ vh
        assert normwise_err(o[:, h].float().cpu().numpy()[rows], ref) < (BF16_TOL if bf16 else F32_TOL)
