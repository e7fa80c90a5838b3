"""Widths that leave the last 256-column tile half or more than half empty: its sums of squares end with the row and do not reach the next one's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P
from oracle import armt_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture
def tile_config():
    yield P.set_gemm_tile_config
    P.set_gemm_tile_config(-1)


@pytest.mark.parametrize("d_model, seg_len", [(128, 512), (320, 512), (384, 1000), (640, 752), (576, 512)])
def test_same_bits(tile_config, d_model, seg_len):
    """Twelve sequences in four layers, 48 cells a launch: the default takes 256 x 256 tiles from 320 columns on, 5 everywhere, 6 takes 128 x 128."""
    shape = S.get_shape("tiny").replace(n_layers=4, d_model=d_model, n_heads=d_model // 64, n_kv_heads=d_model // 64, head_dim=64, d_ff=256, seg_len=seg_len,
                                        n_mem=16, d_mem=32, n_tokens=seg_len * 4, dtype="bf16", mem_k_scale=2.0 ** -6)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = torch.randn(12, shape.n_tokens, d_model, device="cuda", generator=torch.Generator(device="cuda").manual_seed(d_model)).bfloat16()
    got = {}
    for cfg in (6, 5, -1):
        tile_config(cfg)
        got[cfg] = [t.clone() for t in model.forward_batched(x)]
    for a, b, c in zip(got[6], got[5], got[-1]):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b) and torch.equal(a, c)


def test_oracle():
    """One of the sequences of such a launch against the oracle."""
    shape = S.get_shape("tiny").replace(n_layers=2, d_model=384, n_heads=6, n_kv_heads=2, head_dim=64, d_ff=512, seg_len=240, n_mem=16, d_mem=32,
                                        n_tokens=240 * 3, dtype="bf16")
    layers, mem_emb = S.make_weights(shape, seed=0)
    x = S.make_embeddings(shape, seed=0)
    want, _, _ = O.armt_forward_sequential(shape, layers, mem_emb, x)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    xd = model.embed(x)
    hidden, _, _ = model.forward_batched(xd.expand(60, *xd.shape).contiguous())
    err = [float(np.linalg.norm(h.float().cpu().numpy() - want) / np.linalg.norm(want)) for h in (hidden[0], hidden[59])]
    assert max(err) <= 2e-2, err      # the bound of a bf16 pass
