"""The backward passes clear only the parts of their workspace that they have to: what an earlier call left there, NaNs included,
must not show in a result."""
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw, batch, segments", [
    (dict(seg_len=37, n_mem=5), 2, 5),                                                              # fp32, fewer than 16 memory tokens
    (dict(dtype="bf16", d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ff=512, seg_len=100, n_mem=16, d_mem=32), 1, 2),
    (dict(dtype="bf16", d_model=192, n_heads=3, n_kv_heads=1, head_dim=64, d_ff=320, seg_len=61, n_mem=32, d_mem=8, dpfp_nu=4), 2, 18),
])
def test_backward_on_a_used_workspace(kw, batch, segments):
    shape = S.get_shape("tiny").replace(n_layers=3, **kw)
    shape = shape.replace(n_tokens=segments * shape.seg_len)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb)
    gen = torch.Generator(device="cuda").manual_seed(2)
    normal = lambda *dims: torch.randn(*dims, device="cuda", generator=gen)
    x, d_hidden = (normal(batch, shape.n_tokens, shape.d_model).to(model.act_dtype) for _ in range(2))
    *_, tape = model.forward_train(x)
    model.backward(tape, shape.n_tokens, d_hidden)                  # (allocates the workspace)
    got = []
    for byte in (0x00, 0xFF):                                       # zeros, NaNs of either type
        model.bwd_workspace.fill_(byte)
        g = model.backward(tape, shape.n_tokens, d_hidden)
        got.append([t for lw in g["layers"] for t in lw.values()] + [g["mem_emb"], g["x"]])
    for a, b in zip(*got):
        assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("dtype, shift", [("f32", 0), ("bf16", 0), ("bf16", 1)])       # shift: a head that starts 2 bytes past a boundary
@pytest.mark.parametrize("rows, vocab", [(1, 1000), (300, 2050)])
def test_head_backward_on_a_used_workspace(dtype, shift, rows, vocab):
    shape = S.get_shape("tiny").replace(d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ff=512, n_mem=16, dtype=dtype)
    act = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(rows)
    normal = lambda *dims: torch.randn(*dims, device="cuda", generator=gen)
    w = (0.05 * normal(shift + vocab * 256)).to(act)[shift:].view(vocab, 256)
    ends = P.TokenEnds(shape, torch.zeros(1, 256, dtype=act, device="cuda"), normal(256).to(act), w)
    hidden, d_logits = normal(rows, 256).to(act), normal(rows, vocab)
    ends.logits_backward(hidden, d_logits)
    got = []
    for byte in (0x00, 0xFF):
        ends.bws.fill_(byte)
        got.append(ends.logits_backward(hidden, d_logits))
    for a, b in zip(*got):
        assert torch.isfinite(a).all() and torch.equal(a, b)
