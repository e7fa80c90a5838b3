"""fp32 steps whose norms, rotation, feature map and update coefficients run inside the products: both sides of the rules that choose them
(heads of 8, 16, 32 columns or others; d_mem up to 32; at most 16 memory tokens), rows that fill, end inside and fit below a tile, and
widths that cannot be read 16 bytes at a time.  Tolerance of the fp32 configurations (test_gpu_forward.py)."""
import numpy as np
import pytest
import torch

import armt_synth as S
import paper_2506_05229_amd as P
from gpu_util import make_problem, run_hip, run_oracle
from oracle import armt_oracle as O
from test_gpu_forward import _check_f32
from test_gpu_steps import _dev, _memory_problem

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


def test_read_of_many_rows():
    """A long product on more 16-row tiles than CUs takes 32-row tiles: the oracle's values (tolerance of test_gpu_steps.py), and the bits of the
    16-row tiles that a cell by itself takes."""
    g, shape = 3, S.get_shape("tiny").replace(n_layers=3, d_model=1040, n_heads=20, n_kv_heads=5, head_dim=52, seg_len=1387, n_mem=3, d_mem=24,
                                              dpfp_nu=3)
    w, x, _, A, z = _memory_problem(shape, g, np.random.default_rng(3), False)
    steps = P.ArmtSteps(shape)

    def read(cells):
        xd = _dev(x[cells], torch.float32)
        steps.assoc_read(xd, [_dev(w[i]["wm_q"], steps.act_dtype) for i in cells], _dev(A[cells], torch.float32), _dev(z[cells], torch.float32))
        return xd.cpu()

    got = read([0, 1, 2])
    for i in range(g):
        want = O.assoc_read(x[i].astype(np.float64), A[i].astype(np.float64), z[i].astype(np.float64), w[i]["wm_q"].astype(np.float64),
                            shape.assoc_eps, shape.dpfp_nu)
        assert np.abs(got[i].numpy() - want).max() <= 1e-4 * max(1.0, np.abs(want).max())
        assert torch.equal(got[i], read([i])[0])
