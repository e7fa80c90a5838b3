"""Edges of the row kernels of the backward passes: widths that fill, exceed and miss the columns a lane holds in the one-pass norm
backward (and the two-pass one behind it), and vocabularies and row counts that end inside a tile of the converted head gradient."""
import numpy as np
import pytest
import torch

import armt_synth as S
from gpu_util import make_problem, rel_fro
from oracle import armt_oracle_grad as G
from test_gpu_backward import BF16_REL, BF16_REL_MEM, F32_REL, compare, run_hip_grad, upstream
from test_gpu_token_ends import _ends

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,dh", [(1, 34), (1, 36), (4, 64), (5, 52), (8, 64), (5, 104), (10, 104), (24, 86), (28, 110), (41, 100)])
def test_norm_backward_widths(heads, dh):
    d = heads * dh
    shape = S.get_shape("tiny").replace(n_layers=2, d_model=d, n_heads=heads, n_kv_heads=1, head_dim=dh, d_ff=24, seg_len=9, n_mem=3,
                                        d_mem=8, n_tokens=18)
    layers, mem_emb, x = make_problem(shape, seed=5, std=0.02, gain_std=0.1, v_scale=64.0)
    Gs = upstream(shape, 5, with_state=False)
    compare(run_hip_grad(shape, layers, mem_emb, x, Gs, None, True), G.armt_grad(shape, layers, mem_emb, x, *Gs), F32_REL, f"width {d}")


@pytest.mark.parametrize("heads,dh,seg_len", [(12, 64, 520), (24, 128, 128), (32, 128, 112)])
def test_norm_backward_widths_bf16(heads, dh, seg_len):
    """d 768, 3072 and 4096; rows of a chunk that fill and miss the rows a block takes at once (5 of 4, 3 and 2 of 2).  One segment and no gradient into
    the state: random keys of these widths drive gamma of the update through zero, where bf16 sets no bound to the gradient of W_K (1.6e-1 at
    d 768; see test_gpu_backward.py), and the norms are what is compared here."""
    shape = S.get_shape("tiny").replace(dtype="bf16", n_layers=2, d_model=heads * dh, n_heads=heads, n_kv_heads=heads // 4, head_dim=dh, d_ff=64,
                                        seg_len=seg_len, n_mem=16, d_mem=32, n_tokens=seg_len)
    layers, mem_emb, x = make_problem(shape, seed=6, std=0.02, gain_std=0.1)
    Gs = upstream(shape, 6, with_state=False)
    compare(run_hip_grad(shape, layers, mem_emb, x, Gs, None, True), G.armt_grad(shape, layers, mem_emb, x, *Gs), BF16_REL,
            f"bf16 width {heads * dh}", tol_mem=BF16_REL_MEM)


@pytest.mark.parametrize("rows", [1, 63, 65])
@pytest.mark.parametrize("vocab", [301, 1000, 1024, 1027])
def test_head_backward_ragged_bf16(vocab, rows):
    """Tolerance as for the other bf16 head gradients: three bf16 operands, 2e-2."""
    shape = S.get_shape("1b_8k")
    ids, E, gf, W, te = _ends(shape, vocab, 4, shape.seg_len)
    rng = np.random.default_rng(rows)
    h = S.round_to_bf16((rng.standard_normal((rows, shape.d_model)) * 2.0).astype(np.float32))
    Gl = rng.standard_normal((rows, vocab)).astype(np.float32)
    want = G.lm_head_grad(h, gf, W, shape.rms_eps, Gl)
    buf = torch.zeros(rows * vocab + 1, device="cuda")
    for skip in (0, 1):           # the gradient of the logits on and off a 16-byte boundary
        gl = buf[skip:skip + rows * vocab].view(rows, vocab)
        gl.copy_(torch.from_numpy(Gl))
        got = te.logits_backward(torch.from_numpy(h).cuda().to(te.dt), gl)
        torch.cuda.synchronize()
        assert max(rel_fro(a.cpu().numpy(), b) for a, b in zip(got, want)) <= 2e-2
