"""Segments entering and leaving between steps: callers' buffers that do not allow vector accesses, rows whose length is no multiple of four, one segment,
several sequences; the same bits as with aligned buffers and as one sequence at a time."""
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P

pytestmark = pytest.mark.gpu


def shifted(t):
    """The same values, one element behind an aligned address."""
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    out = buf[1:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("segments, change", [
    (1, dict()),
    (3, dict()),
    (3, dict(d_model=122, n_heads=1, n_kv_heads=1, head_dim=122)),
    (2, dict(n_layers=1)),
    (3, dict(d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ff=512, seg_len=112, n_mem=16, d_mem=32, dtype="bf16")),
])
@pytest.mark.parametrize("diagonal", [True, False])
def test_unaligned_buffers(segments, change, diagonal):
    shape = S.get_shape("tiny").replace(**change)
    shape = shape.replace(n_tokens=shape.seg_len * segments)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb, device="cuda:0")
    x = model.embed(S.make_embeddings(shape, seed=2))
    want = [t.clone() for t in model.forward(x, diagonal=diagonal)]
    out = tuple(shifted(t) if i == 0 else t.clone() for i, t in enumerate(want))
    out[0].fill_(float("nan"))
    got = model.forward(shifted(x), diagonal=diagonal, out=out)
    for a, b in zip(got, want):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)
    both = model.forward_batched(torch.stack([x.flip(0), x]), diagonal=diagonal)
    for a, b in zip(both, want):
        assert torch.equal(a[1], b)
