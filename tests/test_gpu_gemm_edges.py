"""Edges of the bf16 GEMM's main loop and epilogue on the GPU: the fewest K
tiles of the 256x256 schedule, and output groups that end inside a wave tile
or straddle the parts of a QKV row."""
import numpy as np
import pytest

from paper_2510_01565_amd import dit, synth, workloads
from harness import (BF16_TOL, F32_TOL, host_params, normwise_err, request_inputs, to_dev, upload_params,
                     workspace)
from test_gpu_step import _oracle_step, _run_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [64, 128, 320])   # 1, 2 and 5 K tiles
@pytest.mark.parametrize("out", ["f32", "bf16"])
def test_linear_256x256_few_k_tiles(K, out):
    """Ragged rows and columns (2313 = 36 x 64 + 9); sampled outputs against fp64 dot products."""
    import torch
    M, N = 6001, 2313
    x = synth.normal(11, "x", (M, K), bf16=True)
    w = synth.normal(11, "w", (N, K), std=0.02, bf16=True)
    b = synth.normal(11, "b", (N,), std=0.02, bf16=True)
    y = torch.full((M, N), float("nan"), dtype=torch.float32 if out == "f32" else torch.bfloat16, device="cuda")
    dit.profile_start()
    dit.dit_linear(M, N, K, dit.DIT_BF16, to_dev(x, torch.bfloat16), to_dev(w, torch.bfloat16),
                   to_dev(b, torch.bfloat16), y, dit.DIT_F32 if out == "f32" else dit.DIT_BF16)
    torch.cuda.synchronize()
    assert "gemm_bf16_256x256" in dit.profile_stop()
    got = y.float().cpu().numpy()
    assert np.isfinite(got).all()
    rng = np.random.default_rng(K)
    ms = np.concatenate([[0, M - 1, M - 1, M - 2], rng.integers(0, M, 2000)])
    ns = np.concatenate([[0, N - 1, 0, N - 9], rng.integers(0, N, 2000)])
    ref = (x[ms].astype(np.float64) * w[ns].astype(np.float64)).sum(axis=1) + b[ns].astype(np.float64)
    # bf16 output: one rounding to 8 significant bits
    assert normwise_err(got[ms, ns], ref) < (F32_TOL if out == "f32" else 2 ** -8)


def test_step_width_not_a_multiple_of_the_wave_tile():
    """Hidden size 640: 48-column wave tiles (288x192) straddle the Q / K and K / V boundaries of a
    QKV row, and the rows of two packed requests of odd sizes end inside 16-row groups."""
    m = workloads.ModelShape(hidden=640, heads=10, head_dim=64, mlp_ratio=4, n_double=1, n_single=1,
                             in_channels=64, text_dim=96)
    cfg, shapes, params = host_params(m, 12)
    grids, n_txt, ts = [(40, 45), (3, 7)], [37, 5], [0.3, 0.8]
    lat, txt = request_inputs(m, grids, n_txt, 12)
    dit.profile_start()
    vel, _, _ = _run_step(m, params, shapes, cfg, grids, n_txt, ts, lat, txt)
    ran = dit.profile_stop()
    assert "gemm_bf16_288x192" in ran, list(ran)
    ref = np.concatenate(_oracle_step(m, params, grids, n_txt, ts, lat, txt))
    assert normwise_err(vel.float().cpu().numpy(), ref) < BF16_TOL


@pytest.mark.parametrize("M,N,K", [
    (1, 1, 8), (33, 31, 24), (32, 32, 16), (65, 130, 72),   # fewer chunks than waves, odd tails
    (40, 70, 2048), (100, 33, 2056), (511, 480, 40),        # below 256 blocks: the last K of 2 chunks per buffer, more
    (512, 512, 8), (1024, 1024, 40), (1025, 1030, 264),     # 256 blocks and more: 1 chunk per buffer
])
def test_linear_f32_tiles(M, N, K):
    """fp32 GEMM at the edges of its tiles and buffer depths, without bias and with an output that is not 16-byte aligned;
    K products of N(0, 1) x N(0, 0.02^2) summed in fp32: each of about K roundings errs by up to 2^-24 of a partial
    sum (scale 0.02 sqrt(K)), they add in quadrature, and the largest of up to 10^6 outputs lies some five times
    further out: error below 4 sqrt(K) 2^-23 of the sums' scale."""
    import torch
    x = synth.normal(13, "x", (M, K))
    w = synth.normal(13, "w", (N, K), std=0.02)
    ref = x.astype(np.float64) @ w.astype(np.float64).T
    y = torch.full((M * N + 1,), float("nan"), dtype=torch.float32, device="cuda")
    dit.dit_linear(M, N, K, dit.DIT_F32, to_dev(x, torch.float32), to_dev(w, torch.float32), None, y[1:], dit.DIT_F32)
    torch.cuda.synchronize()
    got = y[1:].cpu().numpy().reshape(M, N)
    assert np.abs(got - ref).max() <= 2 ** -23 * np.sqrt(K) * 0.02 * np.sqrt(K) * 4 + 1e-9


def test_vt_rows_at_every_alignment():
    """Requests whose rows start at positions 0 .. 3 modulo 4 and elsewhere in 16-key groups, in runs longer
    and shorter than an epilogue group of 32 rows, as image and as text rows (both kinds of block)."""
    m = workloads.ModelShape(hidden=192, heads=3, head_dim=64, mlp_ratio=2, n_double=1, n_single=1,
                             in_channels=64, text_dim=64)
    cfg, shapes, params = host_params(m, 14)
    grids = [(1, 1), (5, 7), (6, 11), (3, 1), (8, 9), (7, 19), (2, 47), (16, 16)]
    n_txt = [65, 0, 70, 33, 40, 67, 98, 3]
    ts = [0.1 * (i + 1) for i in range(len(grids))]
    lat, txt = request_inputs(m, grids, n_txt, 14)
    vel, _, _ = _run_step(m, params, shapes, cfg, grids, n_txt, ts, lat, txt)
    ref = np.concatenate(_oracle_step(m, params, grids, n_txt, ts, lat, txt))
    assert normwise_err(vel.float().cpu().numpy(), ref) < BF16_TOL


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("grids,n_txt", [
    ([(1, 1), (16, 16)], [62, 0]),   # rows 32..61 text at 33..62, row 62 image at 0, row 63 the next request's at 64
    ([(2, 5), (16, 16)], [44, 0]),
    ([(3, 1), (3, 1), (16, 16)], [85, 55, 0]),
])
def test_vt_where_text_rows_run_into_image_rows(grids, n_txt, head_dim):
    """Single blocks whose 32-row groups cross from text to image with ends as far apart as consecutive rows
    would be: every request's velocity against the oracle, on a workspace filled with NaN."""
    import torch
    m = workloads.ModelShape(hidden=256, heads=256 // head_dim, head_dim=head_dim, mlp_ratio=2, n_double=0, n_single=2,
                             in_channels=64, text_dim=64)
    cfg, shapes, params = host_params(m, 15)
    ts = [0.2 * (i + 1) for i in range(len(grids))]
    lat, txt = request_inputs(m, grids, n_txt, 15)
    w = upload_params(params, shapes, torch.bfloat16)
    b = dit.Batch([g[0] for g in grids], [g[1] for g in grids], n_txt, ts)
    ws, nws = workspace(cfg, b)
    ws.fill_(255)
    x, e = to_dev(np.concatenate(lat), torch.bfloat16), to_dev(np.concatenate(txt), torch.bfloat16)
    vel = torch.full_like(x, float("nan"))
    dit.dit_step(cfg, w, b, x, e, vel, ws, nws)
    torch.cuda.synchronize()
    got, off = vel.float().cpu().numpy(), 0
    for r, ref in enumerate(_oracle_step(m, params, grids, n_txt, ts, lat, txt)):
        assert normwise_err(got[off:off + len(ref)], ref) < BF16_TOL, r
        off += len(ref)


def test_linear_f32_more_tiles_than_a_grid_row_holds():
    """65 538 x 257 tiles of 32 x 32: past 2^24 blocks of 256 threads, where one grid dimension ends (the output
    is 69 GB).  Rows and columns at both ends and at random, against fp64."""
    import torch
    M, N, K = 2097201, 8195, 8
    if torch.cuda.mem_get_info()[0] < 4 * M * N + (8 << 30):
        pytest.skip("not enough free device memory")
    gen = torch.Generator(device="cuda").manual_seed(16)
    x = torch.randn((M, K), generator=gen, device="cuda")
    w = torch.randn((N, K), generator=gen, device="cuda")
    y = torch.empty((M, N), device="cuda")
    y.fill_(float("nan"))
    dit.dit_linear(M, N, K, dit.DIT_F32, x, w, None, y, dit.DIT_F32)
    torch.cuda.synchronize()
    rng = np.random.default_rng(16)
    rows = torch.tensor(np.unique(np.concatenate([[0, 1, 31, 32, M - 33, M - 2, M - 1], rng.integers(0, M, 500)]))).cuda()
    ref = x[rows].double() @ w.double().T
    # sums of 8 products of N(0, 1): rounding errors of 2^-24 of partial sums of a few units
    assert (y[rows].double() - ref).abs().max().item() < 8 * 2 ** -24 * ref.abs().max().item()
    cols = torch.tensor(np.unique(np.concatenate([[0, 31, 32, N - 4, N - 1], rng.integers(0, N, 60)]))).cuda()
    for r0 in range(0, M, 1 << 18):
        sl = slice(r0, r0 + (1 << 18))
        err = y[sl][:, cols].double() - x[sl].double() @ w[cols].double().T
        assert err.abs().max().item() < 1e-4, r0
    del y
    torch.cuda.empty_cache()
