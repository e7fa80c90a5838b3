"""The persistent 256 x 256 GEMM tile against the 128 x 128 one, bit for bit (same order of the k-steps): several tiles per workgroup, the fewest
k-tiles it takes, an odd number of them, launches that leave some workgroups a tile less, and the epilogues that the forward pass does not reach."""
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture
def tile_config():
    yield P.set_gemm_tile_config
    P.set_gemm_tile_config(-1)


@pytest.mark.parametrize("g, M, N, K", [
    (1, 256, 256, 192),         # one tile, three k-tiles
    (3, 2064, 4096, 192),       # 384 tiles on 256 workgroups, strip on two M-tiles of each group
    (2, 768, 97 * 256, 448),    # 582 tiles, seven k-tiles
    (1, 33 * 256, 8 * 256, 256),        # 33 M-tiles in five M-groups, the last of five
    (20, 272, 7 * 256, 320),    # 16 waves: a strip behind a single M-tile
    (3, 2064, 4096, 128),       # 16 waves: two k-tiles
])
def test_store(tile_config, g, M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    a, b = ([torch.randn(r, K, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(g)] for r in (M, N))
    out = {}
    for cfg in (6, 5):
        tile_config(cfg)
        out[cfg] = P.grouped_gemm(a, b, [torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(g)])
    for i in range(g):
        assert torch.equal(out[5][i], out[6][i]), i
        rows = slice(M - 48, M)
        want = a[i][rows].float() @ b[i].float().T
        assert (out[5][i][rows].float() - want).norm() <= 2.0 ** -8 * want.norm(), i      # one bf16 rounding of the result


@pytest.mark.parametrize("rows", [256, 1024, 1296, 2320])
def test_head(tile_config, rows):
    """fp32 results with a row scale, whole groups of 1024 rows and what is left of them; the head's backward accumulates in fp32."""
    shape = S.get_shape("tiny").replace(d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ff=512, seg_len=240, n_mem=16, d_mem=32,
                                        n_tokens=240, dtype="bf16")
    gen = torch.Generator(device="cuda").manual_seed(rows)
    normal = lambda *dims: torch.randn(*dims, device="cuda", generator=gen)
    vocab = 4096
    ends = P.TokenEnds(shape, normal(1, 256).bfloat16(), (1 + 0.1 * normal(256)).bfloat16(), (0.02 * normal(vocab, 256)).bfloat16())
    hidden, d_logits = normal(rows, 256).bfloat16(), normal(rows, vocab) / rows
    got = {}
    for cfg in (6, 5):
        tile_config(cfg)
        got[cfg] = [ends.logits(hidden).clone(), *(t.clone() for t in ends.logits_backward(hidden, d_logits))]
    for a, b in zip(got[5], got[6]):
        assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("seg_len, segments", [(240, 3), (512, 3), (1000, 2)])
def test_gradients(tile_config, seg_len, segments):
    """Weight gradients over the slots that a layer has (ranges of the reduction, groups of unequal length), activation gradients with the strip."""
    shape = S.get_shape("tiny").replace(n_layers=3, d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ff=512, seg_len=seg_len, n_mem=16, d_mem=32,
                                        n_tokens=seg_len * segments, dtype="bf16", mem_k_scale=2.0 ** -6)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = model.embed(S.make_embeddings(shape, seed=2))
    gen = torch.Generator(device="cuda").manual_seed(3)
    d_hidden = torch.randn(shape.n_tokens, 256, device="cuda", generator=gen).bfloat16()
    got = {}
    for cfg in (6, 5):
        tile_config(cfg)
        *_, tape = model.forward_train(x)
        out = model.backward(tape, shape.n_tokens, d_hidden)
        got[cfg] = [t.clone() for layer in out["layers"] for t in layer.values()] + [out["mem_emb"].clone(), out["x"].clone()]
    for a, b in zip(got[5], got[6]):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)
