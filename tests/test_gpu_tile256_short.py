"""The persistent 256 x 256 tile with one and two k-tiles, fewer than its copies are ahead, against the 128 x 128 tile, bit for bit."""
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P
from test_gpu_gemm_tiles import test_256_tile_same_bits as same_results, tile_config      # noqa: F401  (fixture)
from test_gpu_tile256_cuts import same_in_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [64, 128])
@pytest.mark.parametrize("g, M, N", [
    (1, 256, 256),              # one tile
    (1, 4352, 4352),            # 289 tiles, the last 34 of M-groups of five
    (3, 2064, 4096),            # 384 tiles on 256 workgroups, a shared strip
    (7, 1040, 6144),            # 672 tiles: two or three a workgroup
    (50, 272, 7 * 256),         # a strip of one M-tile's own
])
def test_store(tile_config, g, M, N, K):      # noqa: F811
    same_results(tile_config, g, M, N, K)


@pytest.mark.parametrize("rows", [1, 64, 65, 124, 128])
def test_head(tile_config, rows):      # noqa: F811
    """Weight gradient of the head over up to 128 rows: 129 M-tiles of three panels, added in place, the last M-tile ragged."""
    shape = S.get_shape("tiny").replace(d_model=768, n_heads=12, n_kv_heads=4, head_dim=64, d_ff=512, n_mem=16, d_mem=32, dtype="bf16")
    gen = torch.Generator(device="cuda").manual_seed(rows)
    normal = lambda *dims: torch.randn(*dims, device="cuda", generator=gen)
    vocab = 128 * 256 + 27
    ends = P.TokenEnds(shape, normal(1, 768).bfloat16(), (1 + 0.1 * normal(768)).bfloat16(), (0.02 * normal(vocab, 768)).bfloat16())
    hidden, d_logits = normal(rows, 768).bfloat16(), normal(rows, vocab) / rows
    same_in_all(tile_config, lambda: ends.logits_backward(hidden, d_logits))


@pytest.mark.parametrize("seg_len, d_model, nu", [(256, 1024, 1), (512, 1024, 2), (752, 1024, 1), (512, 128, 3)])
def test_forward(tile_config, seg_len, d_model, nu):      # noqa: F811
    """The read (residual, copy and sums of squares) of models with 64 and 128 features; gate/up of width 128.  80 cells a launch."""
    shape = S.get_shape("tiny").replace(n_layers=4, d_model=d_model, n_heads=d_model // 64, n_kv_heads=max(1, d_model // 256), head_dim=64, d_ff=1024,
                                        seg_len=seg_len, n_mem=16, d_mem=32, dpfp_nu=nu, n_tokens=seg_len * 4, dtype="bf16", mem_k_scale=2.0 ** -6)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = torch.randn(20, shape.n_tokens, d_model, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seg_len)).bfloat16()
    same_in_all(tile_config, lambda: model.forward_batched(x))
