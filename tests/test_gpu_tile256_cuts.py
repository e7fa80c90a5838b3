"""Launches of the persistent 256 x 256 tile that end inside an M-group, where a launch of 128 x 128 tiles goes on, and groups of unequal length that are
spread over all XCDs: the same bits as 128 x 128 tiles alone."""
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P
from test_gpu_gemm_tiles import test_256_tile_same_bits as same_results, tile_config      # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def same_in_all(tile_config, run):      # noqa: F811
    """-1: cut, 5: 256 x 256 tiles alone, 6: 128 x 128."""
    got = {}
    for cfg in (6, 5, -1):
        tile_config(cfg)
        got[cfg] = [t.clone() for t in run()]
    for a, b, c in zip(got[6], got[5], got[-1]):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b) and torch.equal(a, c)


@pytest.mark.parametrize("g, M, N, K", [
    (2, 528, 512, 192),         # three k-tiles, the fewest
    (1, 4352, 4352, 192),       # 17 x 17 tiles in M-groups of 6, 6 and 5: seven panels of the last one are cut off
])
def test_store(tile_config, g, M, N, K):      # noqa: F811
    same_results(tile_config, g, M, N, K)


def test_head(tile_config):      # noqa: F811
    """17 x 16 tiles in fp32, plain and added to what is there."""
    d, vocab, rows = 4096, 4352, 4352
    shape = S.get_shape("tiny").replace(d_model=d, n_heads=64, n_kv_heads=8, head_dim=64, d_ff=512, n_mem=16, d_mem=32, dtype="bf16")
    gen = torch.Generator(device="cuda").manual_seed(0)
    normal = lambda *dims: torch.randn(*dims, device="cuda", generator=gen)
    ends = P.TokenEnds(shape, normal(1, d).bfloat16(), (1 + 0.1 * normal(d)).bfloat16(), (0.02 * normal(vocab, d)).bfloat16())
    hidden, d_logits = normal(rows, d).bfloat16(), normal(rows, vocab) / rows
    same_in_all(tile_config, lambda: ends.logits_backward(hidden, d_logits))


def test_residual(tile_config):      # noqa: F811
    """Six cells of 2320 x 1280: 270 tiles, M-groups of five and four; four panels of the last one are cut off."""
    shape = S.get_shape("tiny").replace(n_layers=6, d_model=1280, n_heads=20, n_kv_heads=4, head_dim=64, d_ff=1024, seg_len=2304, n_mem=16, d_mem=32,
                                        n_tokens=2304 * 7, dtype="bf16", mem_k_scale=2.0 ** -6)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = model.embed(S.make_embeddings(shape, seed=2))
    same_in_all(tile_config, lambda: model.forward(x, diagonal=True))


@pytest.mark.parametrize("segments", [2, 5])
def test_gradients_spread(tile_config, segments):      # noqa: F811
    """Weight gradients of 2 x 4 tiles: a group's tiles divide among the XCDs; layers with short ranges of the reduction and with none."""
    shape = S.get_shape("tiny").replace(n_layers=4, d_model=512, n_heads=8, n_kv_heads=4, head_dim=64, d_ff=1024, seg_len=240, n_mem=16, d_mem=32,
                                        n_tokens=240 * segments, dtype="bf16", mem_k_scale=2.0 ** -6)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = model.embed(S.make_embeddings(shape, seed=2))
    d_hidden = torch.randn(shape.n_tokens, 512, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).bfloat16()

    def run():
        *_, tape = model.forward_train(x)
        out = model.backward(tape, shape.n_tokens, d_hidden)
        return [t for layer in out["layers"] for t in layer.values()] + [out["mem_emb"], out["x"]]

    same_in_all(tile_config, run)
