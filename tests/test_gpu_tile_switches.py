"""Switch 32 of the tile configuration (memory rows in an M-tile of their own) where a launch is cut into whole rounds and a remainder."""
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P

pytestmark = pytest.mark.gpu


def test_cut_without_strip():
    """18 cells of 1040 x 1024: 360 tiles of 256 x 256, 104 behind the whole round."""
    shape = S.get_shape("tiny").replace(n_layers=2, d_model=1024, n_heads=16, n_kv_heads=4, head_dim=64, d_ff=1024, seg_len=1024, n_mem=16, d_mem=32,
                                        n_tokens=1024 * 3, dtype="bf16", mem_k_scale=2.0 ** -6)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = torch.randn(9, shape.n_tokens, 1024, device="cuda", generator=torch.Generator(device="cuda").manual_seed(0)).bfloat16()
    got = {}
    try:
        for cfg in (-1, 3299):
            P.set_gemm_tile_config(cfg)
            got[cfg] = [t.float() for t in model.forward_batched(x)]
    finally:
        P.set_gemm_tile_config(-1)
    for a, b in zip(got[3299], got[-1]):
        assert (a - b).norm() <= 2e-2 * b.norm()      # the bound of a bf16 pass
