"""The persistent tile that computes the whole strip of 16 rows behind a single M-tile, against the 128 x 128 tile, bit for bit."""
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P
from test_gpu_tile256 import test_gradients as same_gradients, test_store as same_results, tile_config      # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g, M, N, K", [
    (50, 272, 7 * 256, 320),            # 350 tiles on 256 workgroups
    (1, 57 * 256 + 16, 512, 192),       # M-groups of eight, the last of one
])
def test_store(tile_config, g, M, N, K):      # noqa: F811
    same_results(tile_config, g, M, N, K)


def test_gradients(tile_config):      # noqa: F811
    same_gradients(tile_config, 256, 3)


@pytest.mark.parametrize("seg_len, heads, dh", [(256, 16, 64), (256, 8, 128), (512, 16, 64), (512, 8, 128), (752, 16, 64)])
def test_epilogues(tile_config, seg_len, heads, dh):      # noqa: F811
    """80 cells a launch at full steps, 320 to 960 tiles: every epilogue of the forward pass with the next tile's products under it; a strip of one M-tile's own, a
    shared one and none."""
    shape = S.get_shape("tiny").replace(n_layers=4, d_model=1024, n_heads=heads, n_kv_heads=heads // 4, head_dim=dh, d_ff=1024, seg_len=seg_len, n_mem=16,
                                        d_mem=32, n_tokens=seg_len * 4, dtype="bf16", mem_k_scale=2.0 ** -6)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    gen = torch.Generator(device="cuda").manual_seed(seg_len + dh)
    x = torch.randn(20, shape.n_tokens, 1024, device="cuda", generator=gen).bfloat16()
    got = {}
    for cfg in (6, 5):
        tile_config(cfg)
        got[cfg] = [t.clone() for t in model.forward_batched(x)]
    for a, b in zip(got[5], got[6]):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)
