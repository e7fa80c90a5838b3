"""Tile orders and strip shares of the 256 x 256 GEMM tile: the same bits as the 128 x 128 tile (same order of the k-steps), on
sizes where the cut into M-groups, the shares of the 16-row strip, short k-loops and ragged last tiles meet."""
import numpy as np
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
    (1, 272, 256, 64),          # one M-tile with the whole strip, one k-tile
    (2, 528, 512, 128),         # two k-tiles: no steady part of the loop
    (1, 784, 256, 192),
    (3, 1040, 768, 320),        # odd number of k-tiles
    (4, 2320, 2048, 192),       # nine M-tiles + strip in two M-groups, 288 tiles: the last 32 of them as 128 x 128 tiles
    (1, 4352, 4352, 128),       # 17 x 17 tiles, no strip, cut inside an M-group
    (5, 1024, 2560, 256),
])
def test_256_tile_same_bits(tile_config, g, M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = [torch.randn(M, K, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(g)]
    b = [torch.randn(N, K, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(g)]
    out = {}
    for cfg in (6, 5, -1):
        tile_config(cfg)
        out[cfg] = P.grouped_gemm(a, b, [torch.zeros(M, N, device="cuda", dtype=torch.bfloat16) for _ in range(g)])
    for i in range(g):
        want = a[i].float() @ b[i].float().T
        # one bf16 rounding of the result (2^-9) on top of fp32 sums of K products
        assert (out[5][i].float() - want).norm() <= 2.0 ** -8 * want.norm(), i
        assert torch.equal(out[5][i], out[6][i]) and torch.equal(out[-1][i], out[6][i]), i


@pytest.mark.parametrize("seg_len, heads, dh", [(256, 4, 64), (512, 2, 128), (768, 4, 64), (1000, 4, 64), (2304, 4, 64), (2304, 2, 128)])
def test_forward_256_tile_same_bits(tile_config, seg_len, heads, dh):
    """All epilogues (residual, rotary embedding, transposed V, SwiGLU) on cells whose strip lies on 1, 2, 3 and 9 M-tiles."""
    shape = S.get_shape("tiny").replace(n_layers=2, d_model=256, n_heads=heads, n_kv_heads=heads // 2, head_dim=dh, d_ff=512,
                                        seg_len=seg_len, n_mem=16, d_mem=32, n_tokens=seg_len * 3, dtype="bf16")
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = model.embed(S.make_embeddings(shape, seed=2))
    got = []
    for cfg in (6, 5):
        tile_config(cfg)
        got.append([t.clone() for t in model.forward(x, diagonal=True)])
    for a, b in zip(*got):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)


# 7 and 8: the tiles with four k-tiles in LDS that launches of at most one workgroup per CU take
@pytest.mark.parametrize("g, M, N, K", [
    (1, 16, 72, 64),            # less than a tile, one k-tile: fewer than the ring holds
    (2, 80, 256, 128),          # one M-tile of 64 and the strip, two k-tiles
    (3, 144, 384, 192),         # one M-tile of 128 and the strip
    (1, 300, 520, 320),         # ragged in M and N
    (2, 1040, 512, 1024),
])
def test_deep_ring_tiles_same_bits(tile_config, g, M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    a, b = ([torch.randn(r, K, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(g)] for r in (M, N))
    out = {}
    for cfg in (1, 7, 8):
        assert tile_config(cfg) in (-1, 1, 7)
        out[cfg] = P.grouped_gemm(a, b, [torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(g)])
    for i in range(g):
        want = a[i].float() @ b[i].float().T
        assert (out[1][i].float() - want).norm() <= 2.0 ** -8 * want.norm(), i
        assert torch.equal(out[7][i], out[1][i]) and torch.equal(out[8][i], out[1][i]), i


@pytest.mark.parametrize("seg_len, heads, dh", [(50, 4, 64), (112, 2, 128), (300, 4, 64), (1024, 4, 64), (2304, 2, 128)])
def test_forward_deep_ring_tiles_same_bits(tile_config, seg_len, heads, dh):
    """All epilogues of configurations 7 and 8, with and without the strip, on ragged and on whole last M-tiles."""
    shape = S.get_shape("tiny").replace(n_layers=2, d_model=256, n_heads=heads, n_kv_heads=heads // 2, head_dim=dh, d_ff=512,
                                        seg_len=seg_len, n_mem=16, d_mem=32, n_tokens=seg_len * 3, dtype="bf16")
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = model.embed(S.make_embeddings(shape, seed=2))
    got = []
    for cfg in (1, 7, 8):
        tile_config(cfg)
        got.append([t.clone() for t in model.forward(x, diagonal=True)])
    for a, b, c in zip(*got):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b) and torch.equal(a, c)
