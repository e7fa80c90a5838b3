"""fp32 steps whose norms, rotation, feature map and update coefficients run inside the products: both sides of the rules that choose them
(heads of 8, 16, 32 columns or others; d_mem up to 32; at most 16 memory tokens), rows that fill, end inside and fit below a tile, and
widths that cannot be read 16 bytes at a time.  Tolerance of the fp32 configurations (test_gpu_forward.py)."""
import pytest
import torch

import armt_synth as S
from gpu_util import make_problem, run_hip, run_oracle
from test_gpu_forward import _check_f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,dh,seg_len,n_mem,d_mem,nu", [
    (4, 8, 33, 5, 12, 2), (5, 16, 64, 16, 32, 3), (4, 32, 9, 3, 8, 1), (3, 32, 70, 17, 33, 3), (2, 64, 47, 16, 31, 4),
    (1, 34, 31, 1, 1, 1), (3, 22, 65, 15, 32, 8)])
def test_fused_f32_step_matches_oracle(heads, dh, seg_len, n_mem, d_mem, nu):
    shape = S.get_shape("tiny").replace(n_layers=3, d_model=heads * dh, n_heads=heads, n_kv_heads=1, head_dim=dh, d_ff=44, seg_len=seg_len,
                                        n_mem=n_mem, d_mem=d_mem, dpfp_nu=nu, n_tokens=4 * seg_len)
    prob = make_problem(shape, seed=9, std=0.02, gain_std=0.1, v_scale=64.0)
    want = run_oracle(shape, *prob)
    got = {diag: run_hip(shape, *prob, diagonal=diag) for diag in (True, False)}
    for diag, res in got.items():
        _check_f32(res, want, f"{heads}x{dh} T {seg_len}+{n_mem} d_mem {d_mem} diag={diag}")
    for a, b in zip(got[True], got[False]):
        assert torch.equal(torch.as_tensor(a), torch.as_tensor(b))
