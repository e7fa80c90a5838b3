"""Feature map of the read in 32 x 64 tiles (d_mem 64): the same bits as in 128 x 128 tiles, for rows that end in a strip, in a ragged tile and in whole tiles."""
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seg_len, n_mem, d_mem", [(48, 16, 64), (112, 16, 64), (128, 16, 64), (300, 16, 64), (480, 32, 64), (112, 16, 32)])
def test_same_bits(seg_len, n_mem, d_mem):
    shape = S.get_shape("tiny").replace(n_layers=2, d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ff=512, seg_len=seg_len, n_mem=n_mem,
                                        d_mem=d_mem, n_tokens=seg_len * 3, dtype="bf16", mem_k_scale=2.0 ** -6)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = model.embed(S.make_embeddings(shape, seed=2))
    try:
        got = []
        for cfg in (6, 4):      # 4: the other products take their default 64 x 128 tiles
            P.set_gemm_tile_config(cfg)
            got.append([t.clone() for t in model.forward(x, diagonal=True)])
    finally:
        P.set_gemm_tile_config(-1)
    for a, b in zip(*got):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)
