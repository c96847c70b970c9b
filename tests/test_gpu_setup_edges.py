"""The setup that rides on a call's first GEMV, and the V relayout of the
stand-alone attention, at the sizes where their index maps can go wrong."""
import numpy as np
import pytest

import oracle as O
from paper_2510_01565_amd import dit, workloads
from harness import BF16_TOL, F32_TOL, host_params, normwise_err, request_inputs
from test_gpu_kernels import _attn_case
from test_gpu_step import _oracle_step, _run_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tf", [8, 256, 264])  # narrowest; widest inside the GEMV; a launch of its own
def test_timestep_width_and_five_requests(tf):
    """Five requests: two GEMV passes, each with its own timesteps; NaN-filled workspace."""
    import torch
    m = workloads.ModelShape(hidden=128, heads=2, head_dim=64, mlp_ratio=2, n_double=1, n_single=1,
                             in_channels=16, text_dim=32, time_freq_dim=tf)
    cfg, shapes, params = host_params(m, 21)
    grids, n_txt, ts = [(1, 1), (7, 9), (8, 8), (3, 5), (2, 31)], [0, 1, 64, 2, 5], [0.0, 0.2, 0.4, 0.7, 1.0]
    lat, txt = request_inputs(m, grids, n_txt, 21)
    stale = torch.full((64 << 20,), float("nan"), dtype=torch.float32, device="cuda")
    del stale  # the workspace is then carved from memory that holds NaNs
    vel, _, _ = _run_step(m, params, shapes, cfg, grids, n_txt, ts, lat, txt)
    ref = np.concatenate(_oracle_step(m, params, grids, n_txt, ts, lat, txt))
    assert normwise_err(vel.float().cpu().numpy(), ref) < BF16_TOL


@pytest.mark.parametrize("bf16,d", [(True, 128), (True, 64), (False, 64)])
@pytest.mark.parametrize("grids,n_txt", [
    ([(1, 1), (9, 7), (8, 8), (5, 13), (1, 15)], [0, 0, 0, 0, 1]),  # 1, 63, 64, 65 and 16 keys
    ([(11, 13)], [50]),                                            # 193: one key into the fourth tile
])
def test_attention_v_relayout(bf16, d, grids, n_txt):
    got, ref = _attn_case(grids, n_txt, 5, d, bf16, 22)
    assert normwise_err(got, ref) < (BF16_TOL if bf16 else F32_TOL)


def test_modulation_rows_beyond_two_rounds_of_blocks():
    """33 280 modulation rows of 512 in fp32: 4160 blocks against 2048 resident ones, so the GEMV's blocks loop
    evenly; five requests, two passes.  Every block's rows reach the velocity."""
    m = workloads.ModelShape(hidden=512, heads=8, head_dim=64, mlp_ratio=1, n_double=0, n_single=21,
                             in_channels=16, text_dim=32, dtype="f32")
    cfg, shapes, params = host_params(m, 23)
    grids, n_txt, ts = [(1, 2), (2, 2), (1, 1), (1, 3), (2, 1)], [1, 0, 2, 1, 0], [0.1, 0.3, 0.5, 0.7, 0.9]
    lat, txt = request_inputs(m, grids, n_txt, 23)
    vel, _, _ = _run_step(m, params, shapes, cfg, grids, n_txt, ts, lat, txt)
    ref = np.concatenate(_oracle_step(m, params, grids, n_txt, ts, lat, txt))
    assert normwise_err(vel.cpu().numpy(), ref) < F32_TOL
